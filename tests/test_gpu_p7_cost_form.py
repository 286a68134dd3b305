"""GPU parity of P7Viterbi on tables at and beyond the bounds of the cost form
(csrc/p7_fast.hpp): profiles it takes, profiles left to the general kernel
(a score above a bound), and, within one call, sequences it leaves to it
(steep length models, non-scoring residues), bit for bit against the
oracle."""
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


def database(rng, prof, n=400):
    """Short and ordinary sequences, some of non-scoring residues only, some
    rich in the profile's best residues (J opens, some saturate)."""
    L = rng.integers(0, 200, size=n)
    L[: n // 4] = rng.integers(0, 9, size=n // 4)
    L[-3:] = (700, 1111, 2000)
    off = np.zeros(n + 1, np.int64)
    np.cumsum(L, out=off[1:])
    res = rng.integers(0, 32, size=int(off[-1])).astype(np.uint8)
    best = prof["msc"][:20].argmax(0).astype(np.uint8)
    for i in range(n):
        a, b = off[i], off[i + 1]
        if i % 7 == 0:
            res[a:b] = 20 + 7 * (i % 2)
        elif i % 3 == 0 and b > a:
            res[a:b] = np.resize(best, b - a)
    return res, off


def check(hm, prof, rng, plan=None, what=""):
    res, off = database(rng, prof)
    p = hm.P7Profile(torch.from_numpy(prof["msc"]).cuda(), torch.from_numpy(prof["trans"]).cuda(),
                     prof["tbm"])
    db = hm.Database(res, off)
    s, f = hm.p7_score(p, db, plan=plan)
    torch.cuda.synchronize()
    es, ef = oracle.p7_score_db(prof, res, off)
    s, f = s.cpu().numpy(), f.cpu().numpy()
    db.close()
    bad = np.nonzero((s != es) | (f != ef))[0]
    assert bad.size == 0, (what, bad[:5], s[bad[:5]], es[bad[:5]], f[bad[:5]], ef[bad[:5]])
    return ef


@pytest.mark.parametrize("kind", ["usual", "holes", "wide"])
@pytest.mark.parametrize("G,M", [(4, 1), (4, 100), (8, 15), (8, 111), (16, 130), (16, 500),
                                 (32, 200), (32, 1000), (64, 127), (64, 700), (64, 2047)])
def test_tables_within_the_bounds(hm, G, M, kind):
    rng = np.random.default_rng(M * 3 + G)
    prof = tables(rng, M, kind)
    Q = -(-(M + 1) // (2 * G))
    print(f"case p7 cost form G={G} Q={Q} M={M} {kind}", flush=True)
    check(hm, prof, rng, hm.make_plan(G, Q), (G, M, kind))


@pytest.mark.parametrize("what", ["transition", "emission", "tbm_high", "tbm_low", "dm"])
def test_tables_beyond_a_bound(hm, what):
    """One entry past a bound sends the whole call to the general kernel."""
    rng = np.random.default_rng(5)
    for M in (40, 400):
        prof = tables(rng, M, "usual")
        if what == "transition":
            prof["trans"][4, M // 2] = 1
        elif what == "emission":
            prof["msc"][3, M - 1] = 1025
        elif what == "tbm_high":
            prof["tbm"] = 1
        elif what == "tbm_low":
            prof["tbm"] = -4001
        else:
            prof["trans"][5, M // 3] = -32768
            prof["trans"][6, M // 3] = -50
        print(f"case p7 beyond {what} M={M}", flush=True)
        check(hm, prof, rng, None, (what, M))


def test_selected_positions_left_by_the_cost_form(hm):
    """A selection whose records the cost form partly leaves: those are
    scored too, entries outside the selection keep their values."""
    rng = np.random.default_rng(8)
    prof = tables(rng, 90, "usual")
    prof["trans"][4, :] = -1                   # I->I costs 1: short targets are left
    res, off = database(rng, prof)
    p = hm.P7Profile(torch.from_numpy(prof["msc"]).cuda(), torch.from_numpy(prof["trans"]).cuda(),
                     prof["tbm"])
    db = hm.Database(res, off)
    order = db.order()
    n = db.nseq
    pos = np.sort(rng.choice(n, n // 2, replace=False)).astype(np.int32)
    dpos = torch.zeros(n, dtype=torch.int32, device="cuda")
    dpos[:pos.size] = torch.from_numpy(pos).cuda()
    cnt = torch.tensor([pos.size], dtype=torch.int32, device="cuda")
    s = torch.full((n,), 77, dtype=torch.int16, device="cuda")
    f = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    print("case p7 selected, partly left", flush=True)
    hm.p7_score_selected(p, db, dpos, cnt, s, f)
    torch.cuda.synchronize()
    es, ef = oracle.p7_score_db(prof, res, off)
    ids = order[pos]
    rest = np.setdiff1d(np.arange(n), ids)
    s, f = s.cpu().numpy(), f.cpu().numpy()
    assert np.array_equal(s[ids], es[ids]) and np.array_equal(f[ids], ef[ids])
    assert (s[rest] == 77).all() and (f[rest] == 9).all()
    db.close()
