"""The wave kernels' prologue (weights through LDS in the chain's order, noise and controls
in one pass) and step loop (four steps a turn) at their edges: horizons around what one pass
of 512 threads draws (64 steps of 8 samples), the longest of each form, remainders of the
loop, partial blocks, more blocks than compute units, host and device state, context and
context-free entry.  Bars: the parity checks' own for the oracle; the entry
points agree bit for bit."""
import numpy as np
import pytest

import parity_checks as pc
import synth

pytestmark = pytest.mark.gpu

WAVE = 2


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1707_02342_amd import mppi
    mppi.lib()
    return mppi


@pytest.mark.parametrize("K,T,explore", [(1, 1, 0.0), (7, 2, 0.5), (9, 63, 0.0), (64, 64, 0.3), (17, 65, 0.0),
                                         (33, 128, 1.0), (2048, 33, 0.01)])
def test_split_prologue_edges(M, orc, K, T, explore):
    prob = synth.with_(synth.c1_problem(seed=K), K=K, T=T, explore=explore, lam=5.0)
    print(f"split K={K} T={T} explore {explore}", flush=True)
    pc.check_iteration(M, orc, prob, synth.ring_map(), synth.mlp_params(32, 2, bias_scale=0.2), synth.C1_X0,
                       synth.random_controls(T, K, scale=0.2), WAVE, it=3)


@pytest.mark.parametrize("K,T,explore", [(2049, 1, 0.0), (2056, 7, 0.5), (3001, 128, 0.0), (9, 129, 0.3),
                                         (2100, 150, 0.0), (17, 256, 1.0)])
def test_wave_prologue_edges(M, orc, K, T, explore):
    prob = synth.with_(synth.c1_problem(seed=K), K=K, T=T, explore=explore, lam=5.0)
    print(f"wave K={K} T={T} explore {explore}", flush=True)
    pc.check_iteration(M, orc, prob, synth.ring_map(), synth.mlp_params(32, 2, bias_scale=0.2), synth.C1_X0,
                       synth.random_controls(T, K, scale=0.2), WAVE, it=3)


@pytest.mark.parametrize("K,T", [(5, 1), (70, 64), (300, 100), (1920, 128)])
def test_split_inputs_from_host_and_device_agree(M, K, T):
    import torch
    prob = synth.with_(synth.c1_problem(seed=K), K=K, T=T)
    cmap, params = synth.ring_map(), synth.mlp_params(32, 1, bias_scale=0.2)
    U0 = synth.random_controls(T, K, scale=0.2)
    x = torch.tensor(np.asarray(synth.C1_X0, np.float32), device="cuda")
    got = []
    for device in (False, True):
        with M.Controller(prob, cmap, params, schedule=WAVE) as c:
            c.set_controls(U0)
            for _ in range(2):
                if device:
                    M.mppi_iterate_device(c.ctx, x.data_ptr())
                else:
                    c.iterate(synth.C1_X0)
            got.append(c.controls())
    cfg, cost = M.make_config(prob, schedule=WAVE), M.make_cost(prob.cost)
    U = torch.tensor(U0, device="cuda")
    m, p = torch.tensor(cmap.data, device="cuda"), torch.tensor(params, device="cuda")
    for it in range(2):
        M.mppi_iterate_noalloc(cfg, cost, 0, M.current_stream(), m.data_ptr(), cmap.data.shape[0],
                               cmap.data.shape[1], cmap.origin_x, cmap.origin_y, cmap.resolution, 32, p.data_ptr(),
                               x.data_ptr(), it, U.data_ptr())
    got.append(U.cpu().numpy())
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
    assert not np.array_equal(got[0], U0)
