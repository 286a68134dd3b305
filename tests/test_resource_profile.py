"""profiles/resources_tuned_plans.md lists both P7Viterbi kernels of every default
plan, and the comment on block sizes (csrc/p7_fast.hpp) what they spill."""
import os
import re

import pytest

pytest.importorskip("torch")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_p7_kernels():
    import paper_1707_09683_amd as hm
    with open(os.path.join(ROOT, "profiles", "resources_tuned_plans.md")) as fh:
        text = fh.read()
    spilt = {}
    for kernel in ("p7_fast_kernel", "p7_kernel"):
        rows = re.findall(rf"^\| {kernel} \| [\d,]+ \| (\d+) \| (\d+) \| (\d+) \| \d+ \| \d+ \| (\d+) ",
                          text, re.M)
        have = {tuple(map(int, r[:3])): int(r[3]) for r in rows}
        for M in (30, 64, 100, 200, 400, 700, 1000, 1100, 1500, 2047, 2200, 2400, 2815):
            p = hm.p7_default_plan(M)
            assert (p.G, p.Q, p.waves_per_block) in have, (kernel, M)
        spilt[kernel] = {k[1]: v for k, v in have.items() if v}
    assert spilt["p7_kernel"] == {}
    with open(os.path.join(ROOT, "paper_1707_09683_amd", "csrc", "p7_fast.hpp")) as fh:
        comment = fh.read()
    said = re.search(r"p7_fast_kernel spills (\d+) bytes per lane at (\d+) registers and (\d+) at (\d+)",
                     comment.replace("\n// ", " "))
    b0, q0, b1, q1 = map(int, said.groups())
    assert spilt["p7_fast_kernel"] == {q0: b0, q1: b1}
