"""Output maps of a frame step in device and host memory, at the edges of the
ways they take there."""

import numpy as np
import pytest
import torch

from test_gpu_host_maps import _batch, _step

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
