"""A trajectory whose position leaves FP32's range for a few steps and comes back is not
finite, in every schedule: the vehicle drives part of a circle whose far side lies beyond
3.4e38 between steps 20 and 28 of 40 (inside one chunk of 16 steps of the quad tile), and,
started further back, the same circle within the range."""
import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1707_02342_amd import mppi
    mppi.lib()
    return mppi


def path(x0, dt, T):
    """Positions after each step in 64 bits."""
    px, py, th = float(x0[0]), float(x0[1]), float(x0[2])
    out = []
    for _ in range(T):
        px += dt * float(x0[4]) * math.cos(th)
        py += dt * float(x0[4]) * math.sin(th)
        th += dt * float(x0[6])
        out.append((px, py))
    return np.array(out)


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("schedule", [1, 2, 3, 4])
def test_excursion_beyond_the_range(M, schedule, axis):
    T, dt, turn = 40, 1e19, math.pi / 34
    params = synth.mlp_params(32, 0).copy()
    params[6 * 32 + 32 + 32 * 32 + 32:] = 0.0       # the dynamic states stay as they are
    cost = synth.CostParams(w_map=1.0, w_speed=0.0, v_des=0.0)
    for start, finite in ((1.77e38, False), (1.50e38, True)):
        x0 = np.zeros(7, np.float32)
        x0[axis], x0[2], x0[4], x0[6] = start, math.pi / 2 * (1 + axis) - 24 * turn, 1e18, turn / dt
        p = np.abs(path(x0, dt, T)).max(axis=1)
        far = np.flatnonzero(p > np.finfo(np.float32).max)
        assert (far.size == 0) == finite and (finite or (17 <= far[0] and far[-1] < 30))
        prob = synth.with_(synth.c1_problem(seed=0), K=70, T=T, dt=dt, cost=cost)
        with M.Controller(prob, synth.ring_map(), params, schedule=schedule) as c:
            U0 = synth.random_controls(T, 1, scale=0.1)
            c.set_controls(U0)
            S, st = c.iterate(x0, want_costs=True)
            assert np.isfinite(S).all() == finite and np.isinf(S).all() != finite
            assert (st == M.MPPI_OK) == finite
            assert np.array_equal(M.mppi_get_controls(c.ctx, T)[0], U0) != finite
