"""The quad schedule at the sizes where its tile can go wrong: horizons at, before and after
a chunk of 16 steps, one sample and one sample past a tile, exploration samples, each state
of the slip terms (which the kernel leaves out where they cannot count), and trajectories
that stop being finite only in their positions.  Bars: the parity checks' own (costs within
1e-5 relative of the FP64 oracle, the update within 1e-5 of the oracle's on the same costs)."""
import numpy as np
import pytest

import parity_checks as pc
import synth

pytestmark = pytest.mark.gpu

QUAD = 4


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1707_02342_amd import mppi
    mppi.lib()
    return mppi


@pytest.mark.parametrize("K,T,slip,explore", [
    (1, 1, "off", 0.0), (64, 15, "weight", 0.0), (65, 16, "impulse", 0.3), (63, 17, "never", 0.5),
    (130, 32, "weight", 1.0), (257, 33, "impulse", 0.01), (16, 256, "off", 0.25)])
def test_quad_tile_edges(M, orc, K, T, slip, explore):
    terms = {"off": {}, "weight": dict(w_slip=2.0), "impulse": dict(slip_cost=50.0, slip_thresh=0.1),
             "never": dict(slip_cost=50.0, slip_thresh=3.0)}[slip]
    cost = synth.CostParams(w_map=100.0, w_speed=1.0, v_des=6.0, **terms)
    prob = synth.with_(synth.c1_problem(seed=K), K=K, T=T, explore=explore, lam=5.0, cost=cost)
    print(f"quad K={K} T={T} slip {slip} explore {explore}", flush=True)
    pc.check_iteration(M, orc, prob, synth.ring_map(), synth.mlp_params(32, 2, bias_scale=0.2), synth.C1_X0,
                       synth.random_controls(T, K, scale=0.2), QUAD, it=2, impulses=slip == "impulse")


@pytest.mark.parametrize("schedule", [1, QUAD])
def test_positions_that_overflow_late_are_not_finite(M, schedule):
    """v_x = 1e18 held by a network whose output is zero and dt = 1e19: the position passes the
    FP32 range at step 35, and nothing else ever leaves it."""
    params = synth.mlp_params(32, 0).copy()
    params[6 * 32 + 32 + 32 * 32 + 32:] = 0.0
    x0 = np.array([0.0, 0.0, 0.0, 0.0, 1e18, 0.0, 0.0], np.float32)
    cost = synth.CostParams(w_map=1.0, w_speed=0.0, v_des=0.0)
    for T, finite in ((30, True), (40, False), (64, False)):
        prob = synth.with_(synth.c1_problem(seed=0), K=70, T=T, dt=1e19, cost=cost)
        with M.Controller(prob, synth.ring_map(), params, schedule=schedule) as c:
            U0 = synth.random_controls(T, 1, scale=0.1)
            c.set_controls(U0)
            S, st = c.iterate(x0, want_costs=True)
            assert np.isfinite(S).all() == finite and np.isinf(S).all() != finite
            assert (st == M.MPPI_OK) == finite
            U, _ = M.mppi_get_controls(c.ctx, T)
            assert np.array_equal(U, U0) != finite
