"""States and frames at the ends of the memory that holds them: a caller's state
is dense (123 x H x W), the library's planes are padded."""

import ctypes as C
import mmap

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

PARAMS = dict(sigma_P=0.01, huber_k=10.0, init_inv_depth=0.5)


def _before_guard(a):
    """A copy of `a` whose last byte is the last before an unreadable page."""
    page = mmap.PAGESIZE
    n = (a.nbytes + page - 1) // page * page
    m = mmap.mmap(-1, n + page)
    base = C.addressof(C.c_char.from_buffer(m))
    libc = C.CDLL(None, use_errno=True)
    assert libc.mprotect(C.c_void_p(base + n), C.c_size_t(page), 0) == 0
    out = np.frombuffer(m, dtype=a.dtype, count=a.size, offset=n - a.nbytes).reshape(a.shape)
    out[...] = a
    return out, m


@pytest.mark.parametrize("shape", [(5, 33), (3, 64), (2, 129)])
def test_unroll_reads_no_more_than_the_state(shape):
    import paper_2606_03989_amd as pv
    H, W = shape
    p = synth.tiny_pair(3, H=H, W=W, inv_depth=0.5, rotvec=[0.001, -0.002, 0.001], trans=[0.004, -0.002, 0.003])
    K = (p["cam"].fx, p["cam"].fy, p["cam"].cx, p["cam"].cy)
    t = pv.Tracker(H, W, K, **PARAMS)
    t.set_keyframe(p["I_s"], p["normals_s"])
    t.set_sigma_map(np.full(shape, 5e-3, np.float32))
    t.track(p["I_t"], 3)
    state, keep = _before_guard(t.get_state())
    u = pv.Unrolled(H, W, K, n_iters=2, max_frames=1, ckpt_every=1, **PARAMS)
    u.set_keyframe(p["I_s"], p["normals_s"])
    u.set_state(state)
    xi, _ = u.forward(p["I_t"][None].astype(np.float32), np.full(shape, 5e-3, np.float32),
                      float(t.params.sigma_N), 10.0)
    # two iterations on the same frame from the same state
    t.track(p["I_t"], 2)
    # (pose means of at most 258 values below 1, summed in another order)
    want = t.get_state()[:6].astype(np.float64).reshape(6, -1).mean(axis=1)
    assert np.abs(xi[0] - want).max() <= 1e-12


def test_largest_frame_of_the_static_z_buffer():
    # 1024 x 2048: H times the row pitch is exactly the static array's 2^21 entries
    import paper_2606_03989_amd as pv
    H, W = 1024, 2048
    t = pv.Tracker(H, W, (1000.0, 1000.0, W / 2, H / 2), **PARAMS)
    img = np.linspace(0.0, 1.0, H * W, dtype=np.float32).reshape(H, W)
    nrm = np.zeros((H, W, 3), np.float32)
    nrm[..., 2] = -1.0
    t.set_keyframe(img, nrm)
    t.track(img, 0)
    t.set_keyframe(img, nrm, transfer_depth=True, noalloc=True)
