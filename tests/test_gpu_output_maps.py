"""Output maps of a frame step in device and host memory, at the edges of the
ways they take there."""

import ctypes as C

import numpy as np
import pytest
import torch

import synth
from test_gpu_host_maps import PARAMS, _batch, _step

pytestmark = pytest.mark.gpu


# the second sequence's maps lie at the end of the first one's, which one launch for both would write last; the
# third one's at its start, across the two
@pytest.mark.parametrize("shapes", [[(1030, 1027), (9, 131), (64, 67)], [(9, 131), (1030, 1027), (9, 131)]])
def test_overlapping_device_maps_keep_the_order_of_the_sequences(shapes):
    import paper_2606_03989_amd as pv
    b, frames = _batch(shapes)
    state = [b.get_state(i) for i in range(b.n)]
    dev = [torch.full((2, H, W), -1.0, device="cuda") for H, W in shapes]
    _step(b, frames, [(pv.DEVICE, d[0].data_ptr(), d[1].data_ptr()) for d in dev])
    want = [d.cpu().numpy().reshape(2, -1) for d in dev]
    for i, s in enumerate(state):
        b.set_state(i, s)
    n = max(H * W for H, W in shapes)
    one = torch.full((2, n), -1.0, device="cuda")
    torch.cuda.synchronize()
    at = [0 if i != 1 else n - shapes[1][0] * shapes[1][1] for i in range(3)]
    _step(b, frames, [(pv.DEVICE, one[0, a:].data_ptr(), one[1, a:].data_ptr()) for a in at])
    exp = np.full((2, n), -1.0, np.float32)
    for a, w in zip(at, want):
        exp[:, a:a + w.shape[1]] = w
    assert np.array_equal(one.cpu().numpy(), exp)


# on both sides of the size from which a map goes to pinned memory by a copy of its own (2^17 pixels)
@pytest.mark.parametrize("shape", [(3, 65), (256, 511), (256, 512), (517, 641)])
@pytest.mark.parametrize("pinned", [(True, True), (True, False), (False, True), (True, None), (None, True)])
def test_frame_maps_in_pinned_memory(shape, pinned):
    """pinned: per map (inverse depth, variance) pinned or pageable host memory, or None: not asked for."""
    import paper_2606_03989_amd as pv
    H, W = shape
    p = synth.tiny_pair(0, H=H, W=W, inv_depth=0.5, rotvec=[0.001, -0.002, 0.001], trans=[0.004, -0.002, 0.003])
    t = pv.Tracker(H, W, (p["cam"].fx, p["cam"].fy, p["cam"].cx, p["cam"].cy), **PARAMS)
    t.set_keyframe(p["I_s"], p["normals_s"])
    frame = np.ascontiguousarray(p["I_t"], np.float32)
    state = t.get_state()
    r = t.track(frame, 2, out_device=True)
    want = [r[k].cpu().numpy() for k in ("inv_depth", "inv_depth_var")]
    for _ in range(2):   # the second time with the memory that the first one took
        t.set_state(state)
        maps = [torch.full((H, W), -1.0, pin_memory=bool(k)) for k in pinned]
        out = pv.TrackOut(out_where=pv.HOST)
        out.inv_depth, out.inv_depth_var = [m.data_ptr() if k is not None else None for m, k in zip(maps, pinned)]
        assert pv.lib().pixvod_track(t._h, C.c_void_p(frame.ctypes.data), pv.HOST, 2, C.byref(out)) == 0
        for m, k, w in zip(maps, pinned, want):
            assert np.array_equal(m.numpy(), w) if k is not None else bool((m == -1.0).all())


# few large sequences, whose maps are formed by more workgroups each than those of many; 33 sequences: the line
@pytest.mark.parametrize("shapes", [[(1030, 1027)], [(700, 701), (3, 5)], [(40, 67)] * 32, [(40, 67)] * 33])
def test_device_maps_of_few_and_many_sequences(shapes):
    import paper_2606_03989_amd as pv
    b, frames = _batch(shapes)
    dev = [torch.full((2, H, W), -1.0, device="cuda") for H, W in shapes]
    _step(b, frames, [(pv.DEVICE, d[0].data_ptr(), d[1].data_ptr()) for d in dev])
    for i, d in enumerate(dev):
        # inverse depth of the state's log-depth, rounded once to FP32 (half an ulp; two for a libm of another ulp)
        want = np.exp(-b.get_state(i)[6].astype(np.float64))
        assert np.abs(d[0].cpu().numpy() - want).max() <= 2 * 2.0 ** -24 * want.max()
        var = d[1].cpu().numpy()
        assert np.isfinite(var).all() and (var > 0).all()


def _textured(H, W, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.rand((1, 1, H // 16 + 2, W // 16 + 2), device="cuda", generator=g)
    a = torch.nn.functional.interpolate(a, scale_factor=16, mode="bilinear")[0, 0, :H, :W].contiguous()
    n = torch.zeros((H, W, 3), device="cuda")
    n[..., 2] = -1.0
    return a, n


# more floats of maps for host memory than a context pins (2^26): they go through device memory
def test_maps_of_a_frame_beyond_the_pinned_memory():
    import paper_2606_03989_amd as pv
    H, W = 5793, 5795
    img, nrm = _textured(H, W, 1)
    r = []
    for device in (True, False):
        t = pv.Tracker(H, W, (0.9 * W, 0.9 * W, W / 2, H / 2), **PARAMS)
        t.set_keyframe(img, nrm)
        r.append(t.track(img, 1, out_device=device))
        t.close()
    for k in ("inv_depth", "inv_depth_var"):
        assert np.isfinite(r[1][k]).all() and np.array_equal(r[0][k].cpu().numpy(), r[1][k])


def test_maps_of_a_batch_beyond_the_pinned_memory():
    import paper_2606_03989_amd as pv
    shapes = [(4097, 4099), (3, 65), (4097, 4097)]
    pairs = [_textured(H, W, k) for k, (H, W) in enumerate(shapes)]
    r = []
    for where in (pv.DEVICE, pv.HOST):
        b = pv.Batch(shapes, [(0.9 * W, 0.9 * W, W / 2, H / 2) for H, W in shapes], **PARAMS)
        b.set_keyframes(list(range(len(shapes))), [p[0] for p in pairs], [p[1] for p in pairs])
        maps = [torch.full((2, H, W), -1.0, device="cuda" if where == pv.DEVICE else "cpu") for H, W in shapes]
        outs = (pv.TrackOut * b.n)()
        for o, m in zip(outs, maps):
            o.out_where, o.inv_depth, o.inv_depth_var = where, m[0].data_ptr(), m[1].data_ptr()
        torch.cuda.synchronize()
        frames = (C.c_void_p * b.n)(*[p[0].data_ptr() for p in pairs])
        assert pv.lib().pixvod_batch_track(b._h, frames, pv.DEVICE, 1, outs) == 0
        b.close()
        r.append([m.cpu().numpy() for m in maps])
    for d, h in zip(*r):
        assert np.isfinite(h).all() and (h[0] > 0).all() and np.array_equal(d, h)
