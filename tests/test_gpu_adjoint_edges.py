"""The reverse kernels at the edges of their row segments (64 pixels per wave):
ragged crops of the differentiation sequence, one frame of four iterations,
against central differences of the FP64 oracle. Tolerances are those of the
crop test in test_gpu_adjoint.py (1e-3; Huber threshold 2e-2), and the sigma
map is compared as there, entry by entry, here at every pixel. A derivative
along one random direction with a bound relative to its own value is no
criterion at these sizes: at 2x65 its terms cancel to 1/66 of their absolute
sum, which turns the 9e-5 that the FP32 state leaves in the gradient into 2e-3
of the result, for any arithmetic between the stored states."""

import numpy as np
import pytest

import synth
from parity import make_unroll, make_unrolled_oracle, sequence_workload

pytestmark = pytest.mark.gpu


def _crop(H, W, seed=5):
    w = sequence_workload("diff320", 1)
    cam = w["cam"]
    x0, y0 = (cam.W - W) // 2, (cam.H - H) // 2
    crop = lambda a: np.ascontiguousarray(a[y0:y0 + H, x0:x0 + W])  # noqa: E731
    ccam = synth.Camera(H=H, W=W, fx=cam.fx, fy=cam.fy, cx=cam.cx - x0, cy=cam.cy - y0)
    rng = np.random.default_rng(seed)
    sig = (5e-3 * (1.0 + 0.2 * rng.uniform(-1.0, 1.0, (H, W)))).astype(np.float32)
    return dict(cam=ccam, I_s=crop(w["I_s"]), N_s=crop(w["N_s"]), frames=[crop(w["frames"][0])], sigma_map=sig,
                sigma_N=float(np.float32(1e-3)), huber_k=10.0, kw=dict(sigma_P=0.01),
                cxi=rng.normal(size=(1, 6)), crho=(rng.normal(size=(1, H, W)) / (H * W)).astype(np.float32))


@pytest.mark.parametrize("shape", [(2, 63), (3, 64), (2, 65), (4, 129)])
def test_ragged_crop_gradients(shape):
    w = _crop(*shape)
    u = make_unroll(w, 4, 3)
    u.forward(np.stack(w["frames"]).astype(np.float32), w["sigma_map"], w["sigma_N"], w["huber_k"])
    g, gN, gk = u.backward(w["cxi"], w["crho"])
    o = make_unrolled_oracle(w, 4)
    fN, fk = o.d_sigma_N(w["cxi"], w["crho"]), o.d_huber_k(w["cxi"], w["crho"])
    H, W = shape
    fd = np.array([[o.d_sigma_entry(w["cxi"], w["crho"], v, x) for x in range(W)] for v in range(H)])
    err, scale = np.abs(g - fd), np.abs(fd).max()
    print(f"{shape}: sigma map {err.max():.3e} of {scale:.3e}, sigma_N {gN:.9e} / {fN:.9e}, "
          f"huber_k {gk:.9e} / {fk:.9e}", flush=True)
    assert np.all(err <= 1e-3 * scale + 1e-3 * np.abs(fd))
    assert abs(gN - fN) <= 1e-3 * abs(fN)
    assert abs(gk - fk) <= 2e-2 * abs(fk)
