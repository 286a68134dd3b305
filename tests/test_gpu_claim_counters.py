"""Records claimed from sixteen counters (one per 1/16 of the blocks), which calls
of many short rows use: each sequence is scored once and exactly, for grids
of fewer blocks than counters and of blocks that do not divide among them.
The workspace's counters tell how many were in use."""
import numpy as np
import pytest

import oracle
from oracle import quant as oq
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M = 40
# workspace: 256 bytes, a 160 KiB image, 131,008 records of 32 bytes, then the
# counters, 128 bytes apart
COUNTERS = 256 + 160 * 1024 + 131_008 * 32


@pytest.fixture(scope="module")
def hm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_09683_amd as m
    return m


@pytest.mark.parametrize("filt", ["msv", "ssv"])
@pytest.mark.parametrize("G,Q,w,blocks", [(64, 1, 16, 13), (64, 1, 16, 17), (64, 1, 8, 33),
                                          (32, 1, 8, 31), (8, 3, 8, 40), (1, 21, 8, 16)])
def test_sixteen_counters(hm, filt, G, Q, w, blocks):
    N = blocks * w * (64 // G)
    rng = np.random.default_rng(N)
    n = max(20000, 8 * N + 3)
    L = rng.integers(1, 17, n)
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
    emis = synth.sample_emissions(rng, M)
    synth.implant(rng, res, off, [emis], 0.1)
    exp = oracle.score_db(filt, oq.quantize(emis, synth.BG), res, off)
    prof = hm.Profile.from_emissions(emis, synth.BG)
    gdb = hm.Database(res, off)
    ws = hm.new_workspace("cuda", n)
    sdt = torch.uint8 if filt == "msv" else torch.int8
    s = torch.full((n,), 99, dtype=sdt, device="cuda")
    f = torch.full((n,), 99, dtype=torch.uint8, device="cuda")
    print(f"case counters {filt} {G}:{Q}:{w} blocks={blocks} n={n}", flush=True)
    (hm.msv_score if filt == "msv" else hm.ssv_score)(prof, gdb, s, f, workspace=ws,
                                                      plan=hm.make_plan(G, Q, w, blocks))
    torch.cuda.synchronize()
    gdb.close()
    used = ws[COUNTERS:COUNTERS + 16 * 128].view(torch.int32).cpu().numpy()[::32]
    assert (used > 0).sum() == min(16, blocks), used
    # at least what is neither a group's first three nor claimed past the end
    assert used.sum() >= n - 3 * N
    bad = np.nonzero((s.cpu().numpy() != exp[0]) | (f.cpu().numpy() != exp[1]))[0]
    assert bad.size == 0, bad[:5]
