"""P7Viterbi's record claims: every record scored once and exactly, for counts
around the number of lane groups, records of 0 to 64 rows (claims are made
with at most 48 rows left) and grids of fewer blocks than claim counters."""
import numpy as np
import pytest

import oracle
from oracle import p7 as op7
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M = 20


@pytest.fixture(scope="module")
def hm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_09683_amd as m
    return m


@pytest.mark.parametrize("G,blocks", [(4, 1), (8, 3), (16, 17), (64, 2)])
def test_every_record_once(hm, G, blocks):
    rng = np.random.default_rng(G)
    emis = synth.sample_emissions(rng, M)
    trans = synth.sample_transitions(rng, M)
    oprof = op7.quantize(emis, trans, synth.BG)
    prof = hm.P7Profile.from_probabilities(emis, trans, synth.BG)
    groups = blocks * 2 * 64 // G
    plan = hm.make_plan(G, -(-(M + 1) // (2 * G)), waves_per_block=2, blocks=blocks)
    for n in (1, groups - 1, groups, groups + 1, 2 * groups + 3, 5 * groups):
        n = max(n, 1)
        L = rng.integers(0, 65, n)
        L[0] = 300
        off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
        res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
        print(f"case G={G} blocks={blocks} n={n}", flush=True)
        gdb = hm.Database(res, off)
        s = torch.full((n,), 12345, dtype=torch.int16, device="cuda")
        f = torch.full((n,), 77, dtype=torch.uint8, device="cuda")
        hm.p7_score(prof, gdb, s, f, plan=plan)
        torch.cuda.synchronize()
        es, ef = oracle.p7_score_db(oprof, res, off)
        assert np.array_equal(s.cpu().numpy(), es), n
        assert np.array_equal(f.cpu().numpy(), ef), n
        gdb.close()
