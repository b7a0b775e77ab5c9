"""The passes at the edges of their row segments (64 pixels per wave, two
waves per SIMD, message information in LDS) and the pose maps away from their
series: one iteration from an identical FP32 state against the oracle, for both
schedules. Tolerance: the parity rule of tests/parity.py (1e-5 of a plane's
largest magnitude, or twice the oracle's own spread at FP32 storage)."""

import numpy as np
import pytest

import synth
from parity import (check_iteration, from_oracle, iteration_spread, make_oracle, make_tracker, plane_errors,
                    to_oracle, tree_from_oracle, tree_to_oracle)

pytestmark = pytest.mark.gpu


def _workload(H, W, seed=3):
    p = synth.tiny_pair(seed, H=H, W=W)
    return dict(cam=p["cam"], I_s=p["I_s"], N_s=p["normals_s"], frames=[p["I_t"]], iters=8,
                kw=dict(init_inv_depth=0.4, huber_k=10.0, sigma_P=0.1))


def _one_iteration(w, schedule, label, setup=None):
    frame = w["frames"][0]
    o = make_oracle(w)
    if setup is not None:
        setup(o)
    o.track(frame, 3)
    s32 = from_oracle(o.get_state())
    t = make_tracker(w, schedule)
    if setup is not None:
        setup(t)
    t.track(frame, 0)
    t.set_state(s32)
    t.iterate(1)
    o.set_state(to_oracle(s32))
    o.set_frame(frame)
    o.iterate(1)
    err = plane_errors(t.get_state(), from_oracle(o.get_state()))
    check_iteration(err, iteration_spread(w, s32, frame, setup=setup), label)


@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("shape", [(2, 63), (3, 64), (2, 65), (5, 128), (4, 129), (2, 193)])
def test_row_segment_edges(shape, schedule):
    _one_iteration(_workload(*shape), schedule, f"{shape}/{schedule}")


@pytest.mark.parametrize("theta", [0.09, 0.2, 1.5, 3.0])
def test_pose_maps_away_from_identity(theta):
    """A prior pose turned by theta: the prior's residual, and the poses that it
    pulls, leave the series around the identity."""
    xi = np.array([0.6 * theta, -0.64 * theta, 0.48 * theta, 0.02, -0.01, 0.03])

    def setup(x):
        x.set_prior(xi)

    _one_iteration(_workload(9, 70), 0, f"theta {theta}", setup)


@pytest.mark.parametrize("shape", [(2, 2), (2, 63), (3, 65), (4, 129)])
def test_damped_row_segment_edges(shape):
    w = _workload(*shape)
    w["kw"]["damping"] = 0.3
    _one_iteration(w, 1, f"damped {shape}")


@pytest.mark.parametrize("damping", [0.0, 0.3])
@pytest.mark.parametrize("n", [2, 5])
def test_one_call_equals_single_iterations(n, damping):
    """n iterations in one call (rotated passes) leave the state of n calls of
    one iteration (final passes only), bit for bit."""
    w = _workload(5, 70)
    w["kw"]["damping"] = damping
    states = []
    for calls, iters in ((1, n), (n, 1)):
        t = make_tracker(w, 1 if damping else 0)
        t.track(w["frames"][0], 2)
        for _ in range(calls):
            t.iterate(iters)
        states.append(t.get_state())
    np.testing.assert_array_equal(states[0], states[1])


@pytest.mark.parametrize("shape", [(2, 63), (3, 65), (18, 128), (33, 129), (130, 2)])
def test_quadtree_workgroup_edges(shape):
    """Quadtree: pixel row segments and node levels around multiples of 64,
    levels with missing children; one iteration against the oracle, and one call
    of three iterations equal to three calls of one."""
    w = _workload(*shape)
    frame = w["frames"][0]
    o = make_oracle(w, 1)
    o.track(frame, 3)
    s32 = tree_from_oracle(o.get_state())
    t = make_tracker(w, 0, topology=1)
    t.track(frame, 0)
    t.set_state(s32)
    t.iterate(1)
    o.set_state(tree_to_oracle(s32))
    o.set_frame(frame)
    o.iterate(1)
    spread = iteration_spread(w, s32, frame, topology=1)
    for part, g, r in zip(("pixels", "nodes"), t.get_state(), tree_from_oracle(o.get_state())):
        check_iteration(plane_errors(g, r), spread[part], f"{shape} {part}")
    states = []
    for calls, iters in ((1, 3), (3, 1)):
        t.set_state(s32)
        for _ in range(calls):
            t.iterate(iters)
        states.append(t.get_state())
    for a, b in zip(*states):
        np.testing.assert_array_equal(a, b)
