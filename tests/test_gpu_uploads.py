"""Controls and network parameters are on the device when the call that sets them returns: a
captured control step that is replayed on another stream reads them without an ordering of
its own.  Bit for bit against a second context driven in order on one stream."""
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


@pytest.mark.parametrize("what", ["controls", "dynamics"])
def test_uploads_are_seen_by_a_replay_on_another_stream(M, what):
    import torch
    prob = synth.with_(synth.c1_problem(seed=1), K=256, T=30)
    own, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(own):
        x = torch.tensor(np.asarray(synth.C1_X0, np.float32), device="cuda")
        u0 = torch.zeros(2, device="cuda")
        y, v0 = x.clone(), u0.clone()
        busy = torch.ones(2048, 2048, device="cuda")
        with M.Controller(prob, synth.ring_map(), synth.mlp_params(32, 0)) as c, \
                M.Controller(prob, synth.ring_map(), synth.mlp_params(32, 0)) as d:
            M.mppi_step_device(c.ctx, x.data_ptr(), u0.data_ptr())
            M.mppi_step_device(d.ctx, y.data_ptr(), v0.data_ptr())
            c.controls(), d.controls()          # the first reads set up what later calls use
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=own):
                M.mppi_step_device(c.ctx, x.data_ptr(), u0.data_ptr())
            for i in range(4):
                for _ in range(20):             # some milliseconds of work ahead of the upload
                    busy = torch.clamp(busy @ busy, 0.0, 1.0)
                for q in (c, d):
                    if what == "controls":
                        q.set_controls(synth.random_controls(30, i, scale=0.3))
                    else:
                        q.set_dynamics(synth.mlp_params(32, i + 1))
                with torch.cuda.stream(other):
                    g.replay()
                other.synchronize()
                M.mppi_step_device(d.ctx, y.data_ptr(), v0.data_ptr())
                assert np.array_equal(c.controls(), d.controls()), i
                own.synchronize()
                assert torch.equal(x, y) and torch.equal(u0, v0), i
