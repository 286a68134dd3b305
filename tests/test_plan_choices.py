"""What the comments on the models behind a call's plan (csrc/hmsv_host.cpp) say of
their choices is what the measurements in profiles/plan_choices.csv say."""
import csv
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("kind,said", [
    ("ssv", r"Over (\d+) other calls its choice takes ([\d.]+)% more time on average than the "
            r"fastest plan, (\d+)% at most"),
    ("p7", r"over (\d+) others its choice takes ([\d.]+)% more than the fastest plan on average, "
           r"(\d+)% at most")])
def test_figures(kind, said):
    with open(os.path.join(ROOT, "profiles", "plan_choices.csv"), newline="") as fh:
        rows = [r for r in csv.DictReader(fh) if r["kind"] == kind]
    over = [max(1.0, float(r["us"]) / float(r["best_us"])) - 1.0 for r in rows]
    with open(os.path.join(ROOT, "paper_1707_09683_amd", "csrc", "hmsv_host.cpp")) as fh:
        text = fh.read().replace("\n// ", " ")
    n, mean, most = re.search(said, text).groups()
    assert int(n) == len(rows)
    assert float(mean) == round(100.0 * sum(over) / len(over), 1)
    assert int(most) == round(100.0 * max(over))


def test_batch_plans_can_be_tuned():
    """Candidates for a batch's plans hold at most 32 registers per lane, and every
    plan of the compiled table for batches is one of them."""
    from paper_1707_09683_amd import autotune as at
    table = at.load_table()[at.DEVICE_KEY + ":batch"]
    for filt in ("msv", "ssv"):
        for M, plan in table[filt].items():
            cand = set(at.candidates(filt, int(M), 32))
            assert tuple(plan) in cand and all(c[1] <= 32 for c in cand)
