"""select, p7_score_selected and the pipeline read nothing from a workspace that
they have not written: the same results whatever it holds, on profiles that
the cost form of P7Viterbi takes whole, in part and not at all."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_09683_amd as hm
    rng = np.random.default_rng(4)
    M = 70
    emis, trans = synth.sample_emissions(rng, M), synth.sample_transitions(rng, M)
    L = np.concatenate([[6000, 2500, 0], rng.integers(0, 400, 2500)])
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
    synth.implant(rng, res, off, [emis], 0.2)
    q = hm.p7_quantize(emis, trans, synth.BG)
    p7 = {}
    for kind in ("whole", "part", "none"):
        t = q["trans"].copy()
        t[4, :M - 1] = {"whole": -70, "part": -2, "none": 1}[kind]
        p7[kind] = hm.P7Profile(torch.from_numpy(q["msc"]).cuda(), torch.from_numpy(t).cuda(),
                                q["tbm"])
    return hm, hm.Profile.from_emissions(emis, synth.BG), p7, hm.Database(res, off)


@pytest.mark.parametrize("kind", ["whole", "part", "none"])
@pytest.mark.parametrize("filt", ["msv", "ssv"])
@pytest.mark.parametrize("fill", [1, 2, 0x7f, 0xff, None])
def test_any_contents(setup, filt, kind, fill):
    hm, prof, p7, db = setup
    n = db.nseq
    thr = 190 if filt == "msv" else -60

    def stages(ws, dirty):
        def spoil():
            if dirty:
                if fill is None:
                    ws.random_(0, 256)
                else:
                    ws.fill_(fill)
            else:
                ws.zero_()
        s, f = (hm.msv_score if filt == "msv" else hm.ssv_score)(prof, db)
        spoil()
        pos, cnt = hm.select(db, s, f, filt, thr, workspace=ws)
        torch.cuda.synchronize()
        k = int(cnt)
        ps = torch.full((n,), -5, dtype=torch.int16, device="cuda")
        pf = torch.zeros(n, dtype=torch.uint8, device="cuda")
        spoil()
        hm.p7_score_selected(p7[kind], db, pos, cnt, ps, pf, workspace=ws)
        spoil()
        r = hm.pipeline(filt, prof, p7[kind], db, thr, workspace=ws)
        torch.cuda.synchronize()
        return k, [pos[:k].clone(), ps, pf, r.filter_score, r.filter_flags, r.positions[:k].clone(),
                   r.count, r.p7_score, r.p7_flags]

    print(f"case dirty pipeline {filt} {kind} fill={fill}", flush=True)
    k, want = stages(hm.new_workspace("cuda", n), False)
    k2, got = stages(hm.new_workspace("cuda", n), True)
    assert 50 < k < n and k2 == k
    for a, b in zip(got, want):
        assert torch.equal(a, b)
