"""GPU parity of P7Viterbi's cost form (csrc/p7_fast.hpp) on calls that it scores
itself: tables from its whole range whose I->I costs leave no ordinary
sequence to the general kernel, at every group width; and the bounds that
send a call to the general kernel.  The workspace's head tells which kernel
had the records."""
import numpy as np
import pytest

import oracle
from test_gpu_p7_cost_form import database
from test_p7_cost_form import tables

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_09683_amd as m
    return m


def score(hm, prof, res, off, plan=None):
    """Scores checked against the oracle; the workspace's first 36 words."""
    p = hm.P7Profile(torch.from_numpy(prof["msc"]).cuda(), torch.from_numpy(prof["trans"]).cuda(),
                     prof["tbm"])
    db = hm.Database(res, off)
    ws = hm.new_workspace("cuda", db.nseq)
    s, f = hm.p7_score(p, db, workspace=ws, plan=plan)
    torch.cuda.synchronize()
    es, ef = oracle.p7_score_db(prof, res, off)
    s, f = s.cpu().numpy(), f.cpu().numpy()
    rows = db.table_rows
    db.close()
    bad = np.nonzero((s != es) | (f != ef))[0]
    assert bad.size == 0, (bad[:5], s[bad[:5]], es[bad[:5]])
    return ws[:4 * 36].view(torch.int32).cpu().numpy(), rows


@pytest.mark.parametrize("kind", ["usual", "holes", "wide"])
@pytest.mark.parametrize("G,M", [(4, 1), (4, 7), (4, 100), (4, 127), (8, 15), (8, 111), (8, 255),
                                 (16, 130), (16, 500), (32, 200), (32, 1000), (64, 127), (64, 128),
                                 (64, 700), (64, 2047), (64, 2500)])
def test_scored_by_the_cost_form(hm, G, M, kind):
    rng = np.random.default_rng(M * 5 + G)
    prof = tables(rng, M, kind)
    # no length model is steeper than -64
    prof["trans"][4] = np.minimum(prof["trans"][4], -64)
    res, off = database(rng, prof, 300 if M > 1500 else 400)
    if M > 2047:
        res[(res >= 21) & (res <= 26)] = 20          # the 34-row image does not fit
    print(f"case p7 cost form runs G={G} M={M} {kind}", flush=True)
    aux, rows = score(hm, prof, res, off, hm.make_plan(G, -(-(M + 1) // (2 * G))))
    assert aux[1] == 1 and (aux[8:8 + rows] == 1).all()
    L = np.diff(off)
    assert aux[5] == (L > 0).sum()
    # left over: those without residues, and those whose C falls out of reach, the
    # ones with only non-scoring residues among them: only the cost form's kernel
    # lists these
    silent = sum(1 for a, b in zip(off[:-1], off[1:])
                 if not ((res[a:b] < 20) | ((res[a:b] > 20) & (res[a:b] < 27))).any())
    assert silent > (L == 0).sum()
    assert silent <= aux[4] <= silent + (len(L) // 4 if kind != "usual" else len(L) // 20)


@pytest.mark.parametrize("what", ["transition", "emission", "tbm_high", "tbm_low", "dm"])
def test_bounds_are_seen(hm, what):
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
        res, off = database(rng, prof, 200)
        print(f"case p7 bounds seen {what} M={M}", flush=True)
        aux, rows = score(hm, prof, res, off)
        fine = np.ones(rows, bool)
        fine[3] = what != "emission"
        assert aux[1] == (what == "emission") and (aux[8:8 + rows] == fine).all()
