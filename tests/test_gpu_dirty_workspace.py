"""Calls read nothing from a workspace that they have not written: whatever it
holds, MSV, SSV, P7Viterbi and the pipeline give the same results."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fill", [0, 1, 2, 0x7f, 0xff, None])
def test_any_contents(fill):
    import paper_1707_09683_amd as hm
    rng = np.random.default_rng(2)
    M = 70
    emis, trans = synth.sample_emissions(rng, M), synth.sample_transitions(rng, M)
    L = np.concatenate([[9000, 4000, 0], rng.integers(0, 400, 2500)])
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
    synth.implant(rng, res, off, [emis], 0.2)
    prof = hm.Profile.from_emissions(emis, synth.BG)
    p7 = hm.P7Profile.from_probabilities(emis, trans, synth.BG)
    gdb = hm.Database(res, off)

    def run(ws):
        out = []
        for fn, p in ((hm.msv_score, prof), (hm.ssv_score, prof), (hm.p7_score, p7)):
            if fill is not None:
                ws.fill_(fill)
            out += list(fn(p, gdb, workspace=ws))
        torch.cuda.synchronize()
        return out

    clean = hm.new_workspace("cuda", gdb.nseq)
    want = []
    for fn, p in ((hm.msv_score, prof), (hm.ssv_score, prof), (hm.p7_score, p7)):
        clean.zero_()
        want += list(fn(p, gdb, workspace=clean))
    torch.cuda.synchronize()
    ws = torch.randint(0, 256, clean.shape, dtype=torch.uint8, device="cuda")
    print(f"case fill={fill}", flush=True)
    for a, b in zip(run(ws), want):
        assert torch.equal(a, b)
    gdb.close()
