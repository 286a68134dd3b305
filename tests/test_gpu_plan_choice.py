"""The plan and the cuts that a call chooses for itself, by database size and
lengths: scores against the oracle and against the tuned plan's."""
import numpy as np
import pytest

import oracle
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
