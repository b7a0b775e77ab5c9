"""Output maps in host memory: through pinned memory and, when large, several
copying threads. The maps of a step have to be the bytes that the same step
gives in device memory, wherever they go and however the destinations lie."""

import ctypes as C

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

PARAMS = dict(sigma_P=0.01, huber_k=10.0, init_inv_depth=0.5)


def _batch(shapes):
    import paper_2606_03989_amd as pv
    pairs = [synth.tiny_pair(k, H=H, W=W, inv_depth=0.5, rotvec=[0.001, -0.002, 0.001], trans=[0.004, -0.002, 0.003])
             for k, (H, W) in enumerate(shapes)]
    b = pv.Batch(shapes, [(p["cam"].fx, p["cam"].fy, p["cam"].cx, p["cam"].cy) for p in pairs], **PARAMS)
    b.set_keyframes(list(range(len(shapes))), [p["I_s"] for p in pairs], [p["normals_s"] for p in pairs])
    return b, [np.ascontiguousarray(p["I_t"], np.float32) for p in pairs]


def _step(b, frames, dst):
    """One frame step of 2 iterations; dst: per sequence (where, inv_depth pointer, inv_depth_var pointer)."""
    import paper_2606_03989_amd as pv
    outs = (pv.TrackOut * b.n)()
    for o, (where, inv, var) in zip(outs, dst):
        o.out_where, o.inv_depth, o.inv_depth_var = where, inv, var
    ptrs = (C.c_void_p * b.n)(*[f.ctypes.data for f in frames])
    assert pv.lib().pixvod_batch_track(b._h, ptrs, pv.HOST, 2, outs) == 0


# one pixel row more than nothing up to several 512 KB chunks and workers (4 MB each)
@pytest.mark.parametrize("shapes", [[(2, 2), (3, 65)], [(9, 131), (1030, 1027), (512, 512)]])
def test_batch_maps_in_host_memory(shapes):
    import paper_2606_03989_amd as pv
    b, frames = _batch(shapes)
    state = [b.get_state(i) for i in range(b.n)]

    def reset():
        for i, s in enumerate(state):
            b.set_state(i, s)

    dev = [torch.full((2, H, W), -1.0, device="cuda") for H, W in shapes]
    _step(b, frames, [(pv.DEVICE, d[0].data_ptr(), d[1].data_ptr()) for d in dev])
    want = [d.cpu().numpy() for d in dev]
    assert all(np.isfinite(w).all() and (w[0] > 0).all() for w in want)

    # every map in host memory
    reset()
    host = [np.full((2, H, W), -1.0, np.float32) for H, W in shapes]
    _step(b, frames, [(pv.HOST, h[0].ctypes.data, h[1].ctypes.data) for h in host])
    for h, w in zip(host, want):
        assert np.array_equal(h, w)

    # some maps, in both memories
    reset()
    host = [np.full((2, H, W), -1.0, np.float32) for H, W in shapes]
    dev[0].fill_(-1.0)
    torch.cuda.synchronize()
    _step(b, frames, [(pv.DEVICE, None, dev[0][1].data_ptr())] +
          [(pv.HOST, h[0].ctypes.data if i % 2 else None, None if i % 2 else h[1].ctypes.data)
           for i, h in list(enumerate(host))[1:]])
    assert np.array_equal(dev[0][1].cpu().numpy(), want[0][1]) and (dev[0][0] == -1.0).all()
    for i, (h, w) in list(enumerate(zip(host, want)))[1:]:
        assert np.array_equal(h[1 - i % 2], w[1 - i % 2]) and (h[i % 2] == -1.0).all()

    # destinations that overlap: written in order, the last one stays
    reset()
    n = max(H * W for H, W in shapes)
    one = np.full(n, -1.0, np.float32)
    _step(b, frames, [(pv.HOST, one.ctypes.data, one.ctypes.data) for _ in shapes])
    exp = np.full(n, -1.0, np.float32)
    for w in want:
        for m in w:
            exp[:m.size] = m.reshape(-1)
    assert np.array_equal(one, exp)


@pytest.mark.parametrize("shape", [(2, 2), (1030, 1027)])
def test_frame_maps_in_host_memory(shape):
    import paper_2606_03989_amd as pv
    H, W = shape
    p = synth.tiny_pair(0, H=H, W=W, inv_depth=0.5, rotvec=[0.001, -0.002, 0.001], trans=[0.004, -0.002, 0.003])
    K = (p["cam"].fx, p["cam"].fy, p["cam"].cx, p["cam"].cy)
    r = []
    for device in (True, False):
        t = pv.Tracker(H, W, K, **PARAMS)
        t.set_keyframe(p["I_s"], p["normals_s"])
        r.append(t.track(p["I_t"], 2, out_device=device))
    for k in ("inv_depth", "inv_depth_var"):
        assert np.array_equal(r[0][k].cpu().numpy(), r[1][k])
    assert np.array_equal(r[0]["xi"], r[1]["xi"]) and r[0]["flags"] == r[1]["flags"]
