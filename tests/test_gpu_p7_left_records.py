"""Which records of a P7Viterbi call the cost form (csrc/p7_fast.hpp) takes: those
whose length model's loop score is no steeper than the profile's smallest
I->I cost, the first of the processing order.  The general kernel runs the
others without a pass through the cost form; each record is scored once and
as the oracle scores it."""
import numpy as np
import pytest

import oracle
from oracle import p7 as op7
from test_p7_cost_form import tables

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_09683_amd as m
    return m


def case(minii, M=60, n=900, lo=0, hi=330):
    rng = np.random.default_rng(minii + 7 * M)
    prof = tables(rng, M, "usual")
    prof["trans"][4] = -np.maximum(minii, rng.integers(0, 90, M))
    prof["trans"][4, M // 2] = -minii
    L = rng.integers(lo, hi, n)
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
    return prof, res, off


def device(hm, prof, res, off):
    p = hm.P7Profile(torch.from_numpy(prof["msc"]).cuda(), torch.from_numpy(prof["trans"]).cuda(),
                     prof["tbm"])
    return p, hm.Database(res, off)


def taken(minii, off):
    """Records with |loop| <= the smallest I->I cost."""
    return sum(1 for L in np.diff(off) if L > 0 and -op7.length_model(int(L))["NN"] <= minii)


@pytest.mark.parametrize("minii", [0, 1, 2, 5, 12, 33, 63, 64, 200])
def test_whole_database(hm, minii):
    prof, res, off = case(minii)
    p, db = device(hm, prof, res, off)
    ws = hm.new_workspace("cuda", db.nseq)
    print(f"case left records I->I {minii}", flush=True)
    s, f = hm.p7_score(p, db, workspace=ws)
    torch.cuda.synchronize()
    es, ef = oracle.p7_score_db(prof, res, off)
    assert np.array_equal(s.cpu().numpy(), es) and np.array_equal(f.cpu().numpy(), ef)
    aux = ws[:32].view(torch.int32).cpu().tolist()
    # {-, within the bounds, smallest I->I, -, left to the general kernel, taken}
    assert aux[1] == 1 and aux[2] == minii
    assert aux[5] == taken(minii, off)
    assert aux[4] == db.nseq - aux[5]


@pytest.mark.parametrize("order", ["longest first", "any"])
@pytest.mark.parametrize("count", [0, 1, 255, 256, 257, 700, 10 ** 6, -3])
def test_selections(hm, order, count):
    minii = 3
    prof, res, off = case(minii, n=1000)
    p, db = device(hm, prof, res, off)
    n = db.nseq
    rng = np.random.default_rng(count & 1023)
    k = max(0, min(count, n))
    pos = rng.choice(n, k, replace=False).astype(np.int32)
    if order == "longest first":
        pos.sort()
    dpos = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    dpos[:k] = torch.from_numpy(pos).cuda()
    cnt = torch.tensor([count], dtype=torch.int32, device="cuda")
    s = torch.full((n,), 77, dtype=torch.int16, device="cuda")
    f = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    ws = hm.new_workspace("cuda", n)
    print(f"case selection {order} {count}", flush=True)
    hm.p7_score_selected(p, db, dpos, cnt, s, f, workspace=ws)
    torch.cuda.synchronize()
    es, ef = oracle.p7_score_db(prof, res, off)
    ids = db.order()[pos]
    rest = np.setdiff1d(np.arange(n), ids)
    s, f = s.cpu().numpy(), f.cpu().numpy()
    assert np.array_equal(s[ids], es[ids]) and np.array_equal(f[ids], ef[ids])
    assert (s[rest] == 77).all() and (f[rest] == 9).all()
    aux = ws[:32].view(torch.int32).cpu().tolist()
    if order == "longest first":
        assert aux[5] == int((pos < taken(minii, off)).sum()) and aux[4] == k - aux[5]
    db.close()
