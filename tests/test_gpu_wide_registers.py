"""Lane groups with more than 32 registers per lane (their scores come through
a ring of chunks): the first and last register counts of each width, remainders
of a chunk, and the table with degenerate residues, bit for bit."""
import numpy as np
import pytest

import oracle
from oracle import quant as oq
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(2, 33), (2, 64), (4, 34), (4, 64), (8, 35), (8, 64), (16, 36), (16, 63), (16, 64),
          (32, 33), (32, 60)]


@pytest.fixture(scope="module")
def hm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_09683_amd as m
    return m


@pytest.mark.parametrize("filt", ["msv", "ssv"])
@pytest.mark.parametrize("degen", [False, True], ids=["plain", "degenerate"])
@pytest.mark.parametrize("gq", SHAPES, ids=lambda t: f"G{t[0]}Q{t[1]}")
def test_wide_register_kernels(hm, filt, degen, gq):
    G, Q = gq
    if degen and G * Q > 1280:                      # the most that 27 table rows allow
        Q = 1280 // G
    M = 2 * G * Q - 1                               # the most that the kernel holds
    rng = np.random.default_rng(M)
    emis = synth.sample_emissions(rng, M)
    n = 400 if M < 1000 else 150
    L = np.concatenate([[1, 2, 15, 16, 17, 2 * M + 700], rng.integers(3, 500, n)])
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
    synth.implant(rng, res, off, [emis], 0.2)
    if degen:
        at = rng.integers(0, len(res), 300)
        res[at] = 21 + at % 6
    exp = oracle.score_db(filt, oq.quantize(emis, synth.BG), res, off)
    prof = hm.Profile.from_emissions(emis, synth.BG)
    gdb = hm.Database(res, off)
    for wpb in (1, 16):
        print(f"case {filt} G={G} Q={Q} M={M} wpb={wpb} degen={degen}", flush=True)
        s, f = (hm.msv_score if filt == "msv" else hm.ssv_score)(
            prof, gdb, plan=hm.make_plan(G, Q, waves_per_block=wpb))
        torch.cuda.synchronize()
        bad = np.nonzero((s.cpu().numpy() != exp[0]) | (f.cpu().numpy() != exp[1]))[0]
        assert bad.size == 0, bad[:5]
    gdb.close()
