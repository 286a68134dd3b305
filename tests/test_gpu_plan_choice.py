"""The plan and the cuts that a call chooses for itself, by database size and
lengths: scores against the oracle and against the tuned plan's."""
import numpy as np
import pytest

import oracle
from oracle import p7 as op7
from oracle import quant as oq
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# sequences, shortest and longest of most, the long ones
SETS = {
    "one": (1, 5, 900, []),
    "few": (60, 1, 300, []),
    "few-long": (40, 10, 60, [9000, 4000]),
    "some": (900, 20, 400, [12000, 3000, 2999]),
    "many-short": (20000, 1, 50, []),
    "many": (6000, 30, 300, [5000] * 5),
}


@pytest.fixture(scope="module")
def hm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_09683_amd as m
    return m


@pytest.mark.parametrize("M", [20, 150, 700, 2400])
@pytest.mark.parametrize("name", list(SETS))
def test_chosen_plan(hm, name, M):
    n, lo, hi, long = SETS[name]
    rng = np.random.default_rng(M + n)
    L = np.concatenate([np.asarray(long, np.int64), rng.integers(lo, hi, n)])
    if M > 1000:
        L = L[:1500]
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
    emis = synth.sample_emissions(rng, M)
    synth.implant(rng, res, off, [emis], 0.1)
    prof = hm.Profile.from_emissions(emis, synth.BG)
    gdb = hm.Database(res, off)
    for filt, fn in (("msv", hm.msv_score), ("ssv", hm.ssv_score)):
        plan = hm.db_default_plan(gdb, filt, M)
        print(f"case {name} {filt} M={M} plan={plan.as_tuple()} "
              f"split={hm.split_info(filt, M, gdb)}", flush=True)
        exp = oracle.score_db(filt, oq.quantize(emis, synth.BG), res, off)
        for p in (None, plan, hm.plan_for(filt, M)):
            s, f = fn(prof, gdb, plan=p)
            torch.cuda.synchronize()
            s, f = s.cpu().numpy(), f.cpu().numpy()
            bad = np.nonzero((s != exp[0]) | (f != exp[1]))[0]
            assert bad.size == 0, (filt, p and p.as_tuple(), bad[:5])
    gdb.close()


@pytest.mark.parametrize("filt", ["msv", "ssv"])
def test_ranges_choose_alone(hm, filt):
    """A call on part of the database chooses for that part and writes no
    other score."""
    rng = np.random.default_rng(4)
    M = 300
    off = np.concatenate([[0], np.cumsum(rng.integers(20, 700, 4000))]).astype(np.int64)
    res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
    emis = synth.sample_emissions(rng, M)
    synth.implant(rng, res, off, [emis], 0.1)
    exp = oracle.score_db(filt, oq.quantize(emis, synth.BG), res, off)
    prof = hm.Profile.from_emissions(emis, synth.BG)
    gdb = hm.Database(res, off)
    sdt = torch.uint8 if filt == "msv" else torch.int8
    for first, count in ((0, 1), (0, 50), (1000, 2000), (3990, 10), (0, 4000)):
        s = torch.full((4000,), 77, dtype=sdt, device="cuda")
        f = torch.full((4000,), 77, dtype=torch.uint8, device="cuda")
        print(f"case range {filt} {first}+{count}", flush=True)
        hm.score_range(filt, prof, gdb, first, count, s, f)
        torch.cuda.synchronize()
        s, f = s.cpu().numpy(), f.cpu().numpy()
        done = np.nonzero(f != 77)[0]
        assert len(done) == count
        assert np.array_equal(s[done], exp[0][done]) and np.array_equal(f[done], exp[1][done])
        assert (s[f == 77] == 77).all()
    gdb.close()


@pytest.mark.parametrize("M", [20, 150, 900])
@pytest.mark.parametrize("name", ["one", "few-long", "many-short"])
@pytest.mark.parametrize("degen", [False, True], ids=["plain", "degenerate"])
def test_p7_chosen_plan(hm, name, M, degen):
    n, lo, hi, long = SETS[name]
    rng = np.random.default_rng(M + n)
    L = np.concatenate([np.asarray(long, np.int64) // 4, rng.integers(lo, hi, min(n, 4000))])
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
    if degen:
        res[::7] = 21 + res[::7] % 6
    emis, trans = synth.sample_emissions(rng, M), synth.sample_transitions(rng, M)
    prof = hm.P7Profile.from_probabilities(emis, trans, synth.BG)
    gdb = hm.Database(res, off)
    exp = oracle.p7_score_db(op7.quantize(emis, trans, synth.BG), res, off)
    for p in (None, hm.p7_default_plan(M)):
        print(f"case p7 {name} M={M} {p and p.as_tuple()} degen={degen}", flush=True)
        s, f = hm.p7_score(prof, gdb, plan=p)
        torch.cuda.synchronize()
        assert np.array_equal(s.cpu().numpy(), exp[0])
        assert np.array_equal(f.cpu().numpy(), exp[1])
    gdb.close()


def test_batch_plans(hm):
    """Queries of a batch get plans of at most 32 registers; the scores are
    those of single calls."""
    from paper_1707_09683_amd.batch import Batch
    rng = np.random.default_rng(8)
    L = rng.integers(20, 600, 3000)
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
    gdb = hm.Database(res, off)
    qs = [(f, hm.Profile.from_emissions(synth.sample_emissions(rng, M), synth.BG))
          for f, M in (("msv", 600), ("ssv", 40), ("msv", 2300), ("ssv", 130))]
    b = Batch(qs, gdb)
    b.launch()
    torch.cuda.synchronize()
    for (filt, p), plan, s, f in zip(qs, b.plans, b.scores, b.flags):
        assert plan.Q <= 32 and 2 * plan.G * plan.Q > p.M
        s1, f1 = (hm.msv_score if filt == "msv" else hm.ssv_score)(p, gdb)
        torch.cuda.synchronize()
        assert torch.equal(s, s1) and torch.equal(f, f1)
    b.close()
    gdb.close()
