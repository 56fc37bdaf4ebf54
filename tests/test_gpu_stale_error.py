"""An error that some other HIP call of the thread has left behind does not make a reading
call fail: each reports the result of its own calls."""
import ctypes as C
import re

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def runtimes():
    with open("/proc/self/maps") as f:
        libs = {m.group(1) for m in re.finditer(r"(/\S*libamdhip64\.so\S*)", f.read())}
    assert libs
    return [C.CDLL(path) for path in libs]


def leave_an_error():
    """hipSetDevice of a device that is not there: refused by the host, and remembered."""
    for hip in runtimes():
        assert hip.hipSetDevice(1000) != 0


@pytest.fixture
def cleared():
    """The error does not outlive the test."""
    yield
    for hip in runtimes():
        hip.hipGetLastError()


def test_reads_after_an_unrelated_error(cleared):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1707_02342_amd import mppi as M
    prob = synth.with_(synth.c1_problem(seed=1), K=256, T=30)
    with M.Controller(prob, synth.ring_map(), synth.mlp_params(32, 0)) as c:
        c.iterate(synth.C1_X0)
        U, stats = c.controls(), c.stats()
        for _ in range(3):                          # by copies first, then through pinned memory
            for read in (lambda: np.array_equal(c.controls(), U), lambda: c.stats()[:2] == stats[:2],
                         lambda: c.iteration == 1):
                leave_an_error()
                assert read()
        leave_an_error()
        c.set_controls(U)
