"""The pass of small images (four waves per 64 pixels, up to 256 row segments)
against the one-wave pass, which a batch takes at every size: both have to leave
the same bits, below, at and above the size where a context changes over."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

PARAMS = dict(sigma_P=0.01, huber_k=10.0, init_inv_depth=0.5)


@pytest.mark.parametrize("shape", [(2, 2), (2, 63), (3, 65), (4, 129), (256, 33), (128, 66), (257, 40), (129, 65)])
def test_split_pass_equals_one_wave(shape):
    import paper_2606_03989_amd as pv
    H, W = shape
    p = synth.tiny_pair(3, H=H, W=W, inv_depth=0.5, rotvec=[0.001, -0.002, 0.001], trans=[0.004, -0.002, 0.003])
    K = (p["cam"].fx, p["cam"].fy, p["cam"].cx, p["cam"].cy)
    t = pv.Tracker(H, W, K, **PARAMS)
    t.set_keyframe(p["I_s"], p["normals_s"])
    b = pv.Batch([shape], [K], **PARAMS)
    b.set_keyframes([0], [p["I_s"]], [p["normals_s"]])
    for n in (1, 2, 7):          # the final pass alone, after one and after several passes
        r, q = t.track(p["I_t"], n), b.track([p["I_t"]], n, maps=True)[0]
        assert np.array_equal(t.get_state(), b.get_state(0))
        for k in ("xi", "inv_depth", "inv_depth_var"):
            assert np.array_equal(r[k], q[k])
        assert r["valid_fraction"] == q["valid_fraction"] and r["flags"] == q["flags"]


@pytest.mark.parametrize("shape", [(2, 63), (4, 129), (256, 33), (257, 40)])
def test_recompute_follows_the_forward_pass(shape):
    # the reverse sweep recomputes a segment with its tape: with one and with
    # several checkpoints it goes through the same states, so the gradients agree
    # bit for bit
    import paper_2606_03989_amd as pv
    H, W = shape
    p = synth.tiny_pair(3, H=H, W=W, inv_depth=0.5, rotvec=[0.001, -0.002, 0.001], trans=[0.004, -0.002, 0.003])
    K = (p["cam"].fx, p["cam"].fy, p["cam"].cx, p["cam"].cy)
    rng = np.random.default_rng(0)
    sig = (5e-3 * (1.0 + 0.2 * rng.uniform(-1.0, 1.0, shape))).astype(np.float32)
    cxi, crho = rng.normal(size=(1, 6)), (rng.normal(size=(1, H, W)) / (H * W)).astype(np.float32)
    out = []
    for every in (1, 2, 5):
        u = pv.Unrolled(H, W, K, n_iters=5, max_frames=1, ckpt_every=every, **PARAMS)
        u.set_keyframe(p["I_s"], p["normals_s"])
        u.forward(p["I_t"][None].astype(np.float32), sig, 1e-3, 10.0)
        out.append(u.backward(cxi, crho))
    for g, gN, gk in out[1:]:
        assert np.isfinite(g).all() and np.array_equal(g, out[0][0])
        assert gN == out[0][1] and gk == out[0][2]
