"""The floor under the first D~ of an element (csrc/p7_fast.hpp) is F less the rise
of its own slot: the CPU model of the cost form with that floor equals the
oracle, on profiles of long deletions above all, and completes its delete
chains in fewer passes than with the largest rise of the profile."""
import inspect

import numpy as np
import pytest

import oracle
import test_p7_cost_form as cost


def models():
    """The model with either floor, counting passes of delete chains."""
    src = inspect.getsource(cost.model)
    one = src.replace("            D[first] = np.maximum(D[first], in0)\n",
                      "            passes.append(1)\n            D[first] = np.maximum(D[first], in0)\n")
    assert one != src
    own = one.replace("    L = len(x)\n", """    rises = np.zeros(n, np.int64)
    for s in range(M - 1, 0, -1):
        rises[s] = 0 if sDD[s + 1] == NEG else max(0, rises[s + 1] + sDD[s + 1])
    L = len(x)
""").replace("D[s] = max(inn[s], F - rise)", "D[s] = max(inn[s], F - rises[s])")
    assert "F - rises[s]" in own and "for s in range(M - 1, 0, -1)" in own
    out = []
    for text in (one, own):
        scope = dict(vars(cost), passes=[])
        exec(text, scope)
        out.append(scope)
    return out


@pytest.mark.parametrize("kind", ["usual", "holes", "wide", "long deletes"])
def test_own_rise(kind):
    one, own = models()
    rng = np.random.default_rng(21)
    scored = 0
    for trial in range(30):
        M = int(rng.integers(2, 40))
        G = int(rng.choice([1, 2, 4]))
        Q = -(-(M + 1) // (2 * G)) + int(rng.integers(0, 2))
        prof = cost.tables(rng, M, "usual" if kind == "long deletes" else kind)
        prof["trans"][4] = np.minimum(prof["trans"][4], -64)
        if kind == "long deletes":
            prof["trans"][6, :M - 1] = -rng.integers(0, 6, M - 1)
            prof["trans"][5, :M - 1] = -rng.integers(60, 700, M - 1)
        best = prof["msc"][:20].argmax(0)
        for L in (1, 15, 16, 17, 70):
            x = rng.integers(0, 27, size=L).astype(np.uint8)
            if rng.random() < 0.6:
                # a stretch of the profile's best residues, less a part of it
                x = np.resize(np.delete(best, slice(M // 3, 2 * M // 3)), L).astype(np.uint8)
            got = own["model"](prof, x, G, Q)
            assert got == one["model"](prof, x, G, Q)
            if got is not None:
                assert got == oracle.p7_seq(prof, x), (kind, trial, M, G, Q, L)
                scored += 1
    assert scored > 100
    assert len(own["passes"]) <= len(one["passes"])
    if kind == "long deletes":
        assert len(own["passes"]) < 0.8 * len(one["passes"])
