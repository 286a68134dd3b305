"""The frame of P7Viterbi's cost form (csrc/p7_fast.hpp) only moves up: the
floor F never rises above where the step's start put it, whatever J does."""
import inspect

import numpy as np
import pytest

import test_p7_cost_form as cost


@pytest.mark.parametrize("kind", ["usual", "holes", "wide"])
def test_the_floor_never_rises_within_a_step(kind):
    src = inspect.getsource(cost.model)
    moves = []
    watched = src.replace("up = BASE - F\n", "up = BASE - F; moves.append(up)\n")
    assert watched != src
    scope = dict(vars(cost), moves=moves)
    exec(watched, scope)
    rng = np.random.default_rng(11)
    opened = 0
    for _ in range(25):
        M = int(rng.integers(1, 40))
        prof = cost.tables(rng, M, kind)
        prof["trans"][4] = np.minimum(prof["trans"][4], -64)      # no sequence is given up
        best = prof["msc"][:20].argmax(0)
        for L in (17, 64, 100):
            x = np.resize(best, L).astype(np.uint8)
            x[rng.random(L) < 0.1] = 3
            got = scope["model"](prof, x, 2, -(-(M + 1) // 4))
            opened += got is not None and got[0] > 400
    assert opened > 20 and len(moves) > 200 and min(moves) == 0
