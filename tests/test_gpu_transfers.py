"""Results and inputs that pass through pinned host memory: sizes below, at and above what it
holds, many uploads without a synchronising call, replays of a captured launch, and every
instance of a batch.  All comparisons are bit for bit."""
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


def test_costs_below_and_above_the_pinned_memory(M):
    """S_k depends on the counter (k, t) alone: the first costs of every K are the same."""
    T = 4
    U = synth.random_controls(T, 0, scale=0.2)
    ref = None
    for K in (1 << 18) + 64, (1 << 18) - 1, 70000, 65, 1:
        prob = synth.with_(synth.c1_problem(seed=3), K=K, T=T)
        with M.Controller(prob, synth.ring_map(), synth.mlp_params(32, 0), schedule=4) as c:
            c.set_controls(U)
            S, _ = c.iterate(synth.C1_X0, want_costs=True)
            rho = c.stats()[0]
        ref = S if ref is None else ref
        assert np.array_equal(S, ref[:K]) and np.float32(rho) == S.min()


def test_uploads_wrap_and_keep_their_order(M):
    T = 200                                     # 400 words of controls, 1412 of parameters
    prob = synth.with_(synth.c1_problem(seed=0), K=64, T=T)
    with M.Controller(prob, synth.ring_map(), synth.mlp_params(32, 0)) as c:
        for i in range(60):
            U = synth.random_controls(T, i, scale=0.1)
            c.set_controls(U)
            c.set_dynamics(synth.mlp_params(32, i))
            if i % 7 == 6:
                assert np.array_equal(c.controls(), U)
        c.iteration = 5
        S, _ = c.iterate(synth.C1_X0, want_costs=True)
    with M.Controller(prob, synth.ring_map(), synth.mlp_params(32, 59)) as d:
        d.set_controls(U)
        d.iteration = 5
        assert np.array_equal(d.iterate(synth.C1_X0, want_costs=True)[0], S)


def test_replayed_steps_are_read_back(M):
    """Eager reads and a set_controls between the replays of one captured step."""
    import torch
    prob = synth.with_(synth.c1_problem(seed=1), K=256, T=30)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        x = torch.tensor(synth.C1_X0, device="cuda")
        u0 = torch.zeros(2, device="cuda")
        y, v0 = x.clone(), u0.clone()
        with M.Controller(prob, synth.ring_map(), synth.mlp_params(32, 0)) as c, \
                M.Controller(prob, synth.ring_map(), synth.mlp_params(32, 0)) as d:
            M.mppi_step_device(c.ctx, x.data_ptr(), u0.data_ptr())
            M.mppi_step_device(d.ctx, y.data_ptr(), v0.data_ptr())
            stream.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream):
                M.mppi_step_device(c.ctx, x.data_ptr(), u0.data_ptr())
            for i in range(6):
                if i % 2:
                    U = synth.random_controls(30, i, scale=0.1)
                    c.set_controls(U)
                    d.set_controls(U)
                g.replay()
                M.mppi_step_device(d.ctx, y.data_ptr(), v0.data_ptr())
                assert np.array_equal(c.controls(), d.controls())
                stream.synchronize()
                assert torch.equal(x, y) and torch.equal(u0, v0)


@pytest.mark.parametrize("schedule", [0, 1, 4])
def test_batch_instances_are_read_back(M, schedule):
    Ks, Ts = [65, 256, 1, 700], [30, 1, 17, 64]
    prob = synth.c1_problem(seed=2)
    with M.Batch(prob, Ks, Ts, synth.ring_map(), synth.mlp_params(32, 0), schedule=schedule) as b:
        x0 = np.tile(np.asarray(synth.C1_X0, np.float32), (4, 1))
        Us = [synth.random_controls(t, i, scale=0.1) for i, t in enumerate(Ts)]
        for i, U in enumerate(Us):
            b.set_controls(i, U)
            assert np.array_equal(b.controls(i), U)
        b.iterate(x0)
        after = [b.controls(i) for i in range(4)]
        assert all(not np.array_equal(a, U) for a, U in zip(after, Us))
        b.set_controls(1, Us[1])
        assert np.array_equal(b.controls(1), Us[1]) and np.array_equal(b.controls(3), after[3])
        for i, U in enumerate(Us):              # the same controls again: a second iteration differs
            b.set_controls(i, U)
        b.iterate(x0)
        b.synchronize()
        second = [b.controls(i) for i in range(4)]
        assert all(not np.array_equal(s, a) for s, a in zip(second, after))
    nan = synth.constant_map(float("nan"))
    with M.Batch(prob, Ks, Ts, nan, synth.mlp_params(32, 0), schedule=schedule) as b:
        for i, U in enumerate(Us):
            b.set_controls(i, U)
        b.iterate(x0)
        for i, U in enumerate(Us):
            got, st = M.mppi_batch_get_controls(b.b, i, Ts[i])
            assert st == M.MPPI_E_NONFINITE and np.array_equal(got, U)
