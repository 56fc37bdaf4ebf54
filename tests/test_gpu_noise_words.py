"""The generator's division and square root are Newton steps on the chip's reciprocal
instructions that give the correctly rounded results for every word it can draw: 2e8 draws,
24 for each of the 2^23 values a word's upper bits can take (a value is missed with
probability 4e-11), against the oracle's IEEE division and square root, bit for bit."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_noise_of_every_word(orc):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1707_02342_amd import mppi as M
    prob = synth.with_(synth.c1_problem(), K=1 << 20, T=8, seed=20, sigma2=(1.0, 1.0))
    op = orc.OracleProblem(prob, synth.constant_map(0.0), synth.mlp_params(32, 0))
    with ThreadPoolExecutor(8) as pool, \
            M.Controller(prob, synth.constant_map(0.0), synth.mlp_params(32, 0)) as c:
        for first in range(0, 24, 8):
            wanted = pool.map(lambda it: orc.noise(op, it), range(first, first + 8))
            for it, eps in enumerate(wanted, first):
                print(f"noise of iteration {it}", flush=True)
                assert np.array_equal(c.noise(it).view(np.uint32), eps.view(np.uint32)), it
