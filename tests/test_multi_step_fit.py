"""Which problems a multi-step receding launch serves: on every device size, those whose
rollout blocks and one block for every 16 of them fit one block per compute unit (K = 1920
on 256 units, K = 240 on 32), and always with at least one and no idle merger block."""
import shutil
import subprocess
from pathlib import Path

import pytest

HERE = Path(__file__).resolve().parent
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = tmp_path_factory.mktemp("fit") / "fit"
    subprocess.run([HIPCC, "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", str(HERE.parent / "paper_1707_02342_amd" / "csrc"),
                    str(HERE / "helpers" / "multi_step_fit.cpp"), "-o", str(exe)],
                   check=True, capture_output=True, timeout=300)

    def run(cases):
        out = subprocess.run([str(exe)], input="\n".join("%d %d %d" % c for c in cases), check=True,
                             capture_output=True, text=True).stdout.split("\n")
        return [tuple(int(v) for v in l.split()) for l in out if l]
    return run


@pytest.mark.parametrize("cus", [4, 32, 38, 64, 80, 128, 256, 304])
def test_rule_follows_the_compute_units(rule, cus):
    cases = [(G, T, cus) for G in range(1, 310) for T in (1, 2, 8, 9, 17, 100, 112, 113, 128, 129)]
    largest = 0
    for (G, T, _), (fits, mergers, parts) in zip(cases, rule(cases)):
        groups = -(-G // 16)                        # rows are merged in groups of 16 up to 256 of them
        assert fits == (T <= 128 and G <= 256 and G + groups <= cus)
        assert 1 <= parts <= 16
        if fits:
            assert 1 <= mergers <= parts and G + mergers <= cus
            assert mergers == parts or G + mergers == cus
            largest = max(largest, 8 * G)
    assert largest == {4: 24, 32: 240, 38: 280, 64: 480, 80: 600, 128: 960, 256: 1920, 304: 2048}[cus]
