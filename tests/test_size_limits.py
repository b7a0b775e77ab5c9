"""Frames whose padded planes 32-bit byte offsets do not reach are refused, before
any device use (runs without a GPU)."""

import ctypes as C

import pytest
import torch

H_MAX = 1 << 24   # rows of 2 pixels, padded to 64: 2^30 elements


def _create(kind, H, W):
    import paper_2606_03989_amd as pv
    h, K, p = C.c_void_p(), pv.Intrinsics(2.0, 2.0, 1.0, 1.0), pv.default_params()
    L = pv.lib()
    if kind == "frame":
        return L.pixvod_create(H, W, C.byref(K), C.byref(p), C.byref(h))
    if kind == "batch":
        # beside a small one
        hs, ws, ks = (C.c_int * 2)(4, H), (C.c_int * 2)(4, W), (pv.Intrinsics * 2)(K, K)
        return L.pixvod_batch_create(2, hs, ws, ks, C.byref(p), C.byref(h))
    return L.pixvod_unroll_create(H, W, C.byref(K), C.byref(p), 1, 1, 1, C.byref(h))


@pytest.mark.parametrize("kind", ["frame", "batch", "unroll"])
def test_planes_beyond_32_bit_offsets_are_refused(kind):
    import paper_2606_03989_amd as pv
    assert _create(kind, H_MAX + 1, 2) == pv.EINVAL
    assert b"too large" in pv.lib().pixvod_last_error(None)
    if not torch.cuda.is_available():
        # the largest one passes the checks (and needs a device, with more memory than one has)
        assert _create(kind, H_MAX, 2) == pv.ENODEV
