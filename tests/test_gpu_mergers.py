"""A multi-step receding launch with fewer merger blocks than parts of the merged row, as on
a device with few free compute units: each merger block takes several parts in turn.  Equal
to single steps bit for bit."""
import numpy as np
import pytest

import synth
import test_gpu_receding as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1707_02342_amd import mppi
    mppi.lib()
    return mppi, torch


@pytest.mark.parametrize("K,T,mergers", [(1, 1, 1), (9, 8, 3), (240, 128, 2), (129, 113, 1), (1913, 100, 15),
                                         (1920, 128, 5)])
def test_fewer_mergers_than_parts(env, monkeypatch, K, T, mergers):
    M, torch = env
    monkeypatch.setenv("MPPI_STEP_MERGERS", str(mergers))
    prob = synth.with_(synth.c1_problem(seed=K + T), K=K, T=T, lam=5.0)
    U0 = synth.random_controls(T, K, scale=0.2)
    R._say(f"case: K={K} T={T} mergers={mergers}")
    a = R._run(M, torch, prob, synth.ring_map(), synth.mlp_params(32, 1), synth.C1_X0, U0, 4, True)
    b = R._run(M, torch, prob, synth.ring_map(), synth.mlp_params(32, 1), synth.C1_X0, U0, 4, False)
    for x, y in zip(a[:4], b[:4]):
        np.testing.assert_array_equal(x, y)
    assert np.isfinite(a[0]).all()
