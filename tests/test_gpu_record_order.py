"""Which records a launch's lane groups take, and how split sequences combine:
every sequence is scored once and exactly, for ranges below, at and above one,
two, three and six records per group, with and without long first records."""
import numpy as np
import pytest

import oracle
from oracle import quant as oq
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M = 40


@pytest.fixture(scope="module")
def hm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_09683_amd as m
    return m


def _db(rng, emis, lengths):
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    res = rng.integers(0, 20, int(off[-1])).astype(np.uint8)
    synth.implant(rng, res, off, [emis], 0.1)
    return res, off


def _same(hm, filt, emis, res, off, plan):
    exp = oracle.score_db(filt, oq.quantize(emis, synth.BG), res, off)
    prof = hm.Profile.from_emissions(emis, synth.BG)
    gdb = hm.Database(res, off)
    n = len(off) - 1
    sdt = torch.uint8 if filt == "msv" else torch.int8
    s = torch.full((n,), 99, dtype=sdt, device="cuda")
    f = torch.full((n,), 99, dtype=torch.uint8, device="cuda")
    (hm.msv_score if filt == "msv" else hm.ssv_score)(prof, gdb, s, f, plan=plan)
    torch.cuda.synchronize()
    info = hm.split_info(filt, M, gdb, plan)
    gdb.close()
    bad = np.nonzero((s.cpu().numpy() != exp[0]) | (f.cpu().numpy() != exp[1]))[0]
    assert bad.size == 0, (filt, n, bad[:5])
    return info


@pytest.mark.parametrize("blocks", [1, 2, 17])
@pytest.mark.parametrize("filt", ["msv", "ssv"])
def test_records_per_group(hm, filt, blocks):
    emis = synth.sample_emissions(np.random.default_rng(1), M)
    plan = hm.make_plan(16, 2, waves_per_block=2, blocks=blocks)
    groups = blocks * 2 * 4
    counts = sorted({1, 2, groups - 1, groups, groups + 1, 2 * groups - 1, 2 * groups + 1,
                     3 * groups - 1, 3 * groups, 3 * groups + 1, 5 * groups, 6 * groups,
                     6 * groups + 5, 9 * groups})
    for long in (0, 1, groups // 2):
        for n in counts:
            rng = np.random.default_rng(1000 * n + long)
            L = rng.integers(1, 60, n)
            L[rng.permutation(n)[:min(long, n)]] = rng.integers(150, 250, min(long, n))
            print(f"case {filt} blocks={blocks} n={n} long={long}", flush=True)
            _same(hm, filt, emis, *_db(rng, emis, L), plan)


@pytest.mark.parametrize("filt", ["msv", "ssv"])
@pytest.mark.parametrize("G", [1, 8, 64])
def test_segments_of_long_sequences(hm, filt, G):
    """Split sequences of more segments than are combined at a time (16)."""
    rng = np.random.default_rng(3)
    emis = synth.sample_emissions(rng, M)
    L = np.concatenate([[40000, 24001, 9000, 5000, 4096, 3000, 1000], rng.integers(30, 200, 3000)])
    plan = hm.make_plan(G, -(-(M + 1) // (2 * G)), waves_per_block=4)
    print(f"case {filt} G={G}", flush=True)
    nsplit, nsegs, seg = _same(hm, filt, emis, *_db(rng, emis, L), plan)
    assert nsplit >= 2 and -(-40000 // seg) > 32
