"""A DPP instruction may read a vector register two wait states after a vector instruction
wrote it, and the compiler does not look for that inside inline assembly.  So every block
of the kernels that reads through DPP brings the distance with it: two instructions (or
s_nop 1) ahead of its first DPP read, or at least two inputs of its own that are computed
from the register it reads, so that nothing can be scheduled in between."""
import re
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_1707_02342_amd" / "csrc"


def blocks():
    out = []
    for path in sorted(CSRC.iterdir()):
        if path.suffix not in (".hip", ".h"):
            continue
        src = path.read_text()
        for m in re.finditer(r"asm volatile\(\s*((?:\"[^\"]*\"\s*)+)((?::[^;]*)?)\);", src):
            text = "".join(re.findall(r'"([^"]*)"', m.group(1)))
            if "_dpp" in text:
                out.append((f"{path.name}:{src[:m.start()].count(chr(10)) + 1}", src[:m.start()],
                            [i.strip() for i in text.replace("\\t", "").split("\\n") if i.strip()], m.group(2)))
    return out


def operands(constraints):
    """[(constraint, expression)] in order of their numbers."""
    ops, i = [], 0
    while (m := re.compile(r'"([^"]*)"\(').search(constraints, i)):
        depth, j = 1, m.end()
        while depth:
            depth += {"(": 1, ")": -1}.get(constraints[j], 0)
            j += 1
        ops.append((m.group(1), constraints[m.end():j - 1].strip()))
        i = j
    return ops


def wait_states(instructions):
    n = 0
    for ins in instructions:
        if "_dpp" in ins:
            return n
        n += int(ins.split()[1]) + 1 if ins.startswith("s_nop") else 1
    return n


@pytest.mark.parametrize("where,before,instructions,constraints", blocks(), ids=lambda v: v if isinstance(v, str) and ":" in v and len(v) < 60 else "")
def test_dpp_source_is_two_wait_states_old(where, before, instructions, constraints):
    if wait_states(instructions) >= 2:
        return
    first = next(i for i in instructions if "_dpp" in i)
    ops = operands(constraints)
    source = ops[int(re.findall(r"%(\d+)", first)[1])][1]
    derived = 0
    for kind, expr in ops:
        if kind.startswith("+"):
            assigned = re.findall(r"\b" + re.escape(expr) + r"\s*=\s*([^;]*);", before)
            derived += bool(assigned and re.search(r"\b" + re.escape(source) + r"\b", assigned[-1]))
    assert derived >= 2, f"{where}: {first} may follow the write of {source}"


def test_the_chain_blocks_are_found():
    reads = [sum("_dpp" in i for i in ins) for _, _, ins, _ in blocks()]
    assert reads.count(4) >= 3 and 28 in reads      # layer 1 and the quads' products, a layer 2 product
