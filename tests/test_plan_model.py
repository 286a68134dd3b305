"""The host code that chooses a call's plan, cuts and grid, run without a GPU
(tests/host/model_driver.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1707_09683_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    """Answers of the driver to a list of commands."""
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("driver") / "model_driver")
    p = subprocess.run([hipcc, "-O1", "-std=c++20", "--offload-arch=gfx950",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-w", "-x", "hip",
                        os.path.join(ROOT, "tests", "host", "model_driver.cpp"),
                        os.path.join(CSRC, "select.hip"), "-o", exe],
                       capture_output=True, text=True, timeout=600)
    assert p.returncode == 0, p.stderr[-4000:]

    def ask(commands):
        r = subprocess.run([exe], input="\n".join(commands) + "\n", capture_output=True, text=True,
                           timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        out = r.stdout.strip().split("\n")
        assert len(out) == len(commands) and not any(o.startswith("?") for o in out), out[:3]
        return out
    return ask


@pytest.mark.parametrize("G,w", [(1, 8), (1, 4), (2, 8), (64, 16)])
def test_grid_of_a_plan_holds_no_more_groups_than_records(driver, G, w):
    """A plan's own grid beyond its call's records (2^31 lane groups among
    them): the kernels number three records per lane group in 32 bits."""
    Q = -(-41 // (2 * G))
    per_block = w * (64 // G)
    for n, blocks in ((1, 1), (1, 5), (1000, 3), (1000, 1 << 22), (1000, (1 << 31) - 1),
                      (70000, 100000)):
        got, nsegs, nlong = map(int, driver([f"grid {n} 50 40 {G} {Q} {w} {blocks}"])[0].split())
        assert nsegs == 0
        assert got == min(blocks, -(-n // per_block))
        assert 3 * got * per_block < 1 << 31 and nlong <= got * per_block


@pytest.mark.parametrize("cus", [32, 64, 128])
@pytest.mark.parametrize("kind", [0, 1, 2], ids=["ssv", "msv", "p7"])
def test_part_of_a_gpu_gets_its_own_plan(driver, kind, cus):
    """A partition of the GPU on a database runs as the whole GPU does on as
    many copies of it as there are such partitions: the same width and the same
    cut (the longest record is the same, each SIMD's share too)."""
    k = 256 // cus
    ask = [(M, n) for M in (30, 100, 400, 1000, 2400) for n in (50, 500, 5000)]
    part = driver([f"plan {kind} {M} {cus} {n} 1" for M, n in ask])
    whole = driver([f"plan {kind} {M} 256 {n} {k}" for M, n in ask])
    same = sum(a.split()[0] == b.split()[0] for a, b in zip(part, whole))
    # a segment's record and the launch cost the same on fewer units, so a plan on
    # the edge may differ
    assert same >= len(ask) - 2, list(zip(ask, part, whole))
    # and it is not the whole GPU's plan for that database throughout
    assert part != driver([f"plan {kind} {M} 256 {n} 1" for M, n in ask])


def test_blocks_by_lds(driver):
    """LDS comes in units of 1280 bytes, 128 of them to a CU."""
    for nbytes, blocks in ((1, 128), (1280, 128), (1281, 64), (26880, 6), (32256, 4), (32000, 5),
                           (40960, 4), (40961, 3), (81920, 2), (81921, 1), (163840, 1), (163841, 0)):
        assert int(driver([f"lds {nbytes}"])[0]) == blocks


def test_wavefronts_per_block(driver):
    """Twelve where the image leaves one block to a CU and every lane group has a
    sequence; no more than the kernels are built for."""
    for G, Q, rows, n, cus, waves in ((32, 38, 21, 60000, 256, 12), (32, 38, 21, 6143, 256, 8),
                                      (32, 38, 21, 6144, 256, 12), (32, 38, 21, 768, 32, 12),
                                      (64, 19, 21, 3000, 256, 8), (64, 19, 21, 3072, 256, 12),
                                      (64, 12, 21, 60000, 256, 8), (16, 61, 21, 60000, 256, 12),
                                      (16, 18, 21, 60000, 256, 4), (4, 34, 27, 201525, 256, 8),
                                      (8, 64, 27, 500000, 256, 12)):
        assert int(driver([f"waves {G} {Q} {rows} {n} {cus}"])[0]) == waves, (G, Q, rows, n, cus)
    for G, qmax in ((1, 32), (2, 64), (4, 64), (8, 64), (16, 64), (32, 60), (64, 30)):
        for Q in range(1, qmax + 1):
            for rows in (21, 27):
                w = int(driver([f"waves {G} {Q} {rows} 10000000 256"])[0]) if Q % 7 == 0 else 4
                assert w <= (16 if G >= 32 or Q > 32 else 8)
