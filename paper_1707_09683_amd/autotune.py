"""Autotuner for launch plans: group width and waves per block.

For each filter and each profile length of a grid of M-bins, every valid
plan is timed on a lognormal database sample with HIP events (mean of
back-to-back launches after one warm-up launch) and the fastest is kept.  All candidates must return identical outputs; a plan
that disagrees with the first one fails the run.  Results are written to
``tuned_plans.json`` keyed by the device (architecture and CU count); the
package's ``plan_for()`` reads them.

Run on the GPU:  python -m paper_1707_09683_amd.autotune [--nseq N]

``--choices FILE`` times what a call without a plan chooses for itself (a
model of its time, csrc/hmsv_host.cpp) against every other plan, over
databases of 2,000 to 300,000 sequences, and writes both to a CSV file:
profiles/plan_choices.csv.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
TABLE = os.path.join(HERE, "tuned_plans.json")

M_BINS = (30, 40, 48, 64, 80, 96, 120, 128, 160, 192, 240, 256, 320, 400, 480, 512, 640, 768,
          896, 1000, 1024, 1280, 1536, 1920, 2048, 2400, 3072, 3839)
GROUPS = (1, 2, 4, 8, 16, 32, 64)
WAVES = (2, 3, 4, 5, 6, 8)
# registers per lane the kernels are built for, per group width
QMAX = {1: 32, 2: 64, 4: 64, 8: 64, 16: 64, 32: 60, 64: 30}
LDS_LIMIT = 160 * 1024


def lds_bytes(G, Q):
    """Bytes of a plan's LDS image, as the library computes it."""
    from . import plan_lds_bytes
    return plan_lds_bytes(G, Q)


def q_for(G, M):
    return (M + 1 + 2 * G - 1) // (2 * G)


def candidates(filt, M, qmax=64):
    for G in GROUPS:
        Q = q_for(G, M)
        if Q > min(qmax, QMAX[G]) or lds_bytes(G, Q) > LDS_LIMIT:
            continue
        for wpb in WAVES + ((12, 16) if G >= 32 or Q > 32 else ()):
            yield (G, Q, wpb, 0)


def device_key():
    import torch
    p = torch.cuda.get_device_properties(0)
    arch = getattr(p, "gcnArchName", "unknown").split(":")[0]
    return f"{arch}:{p.multi_processor_count}cu"


def load_table():
    if not os.path.exists(TABLE):
        return {}
    with open(TABLE) as fh:
        return json.load(fh)


def lookup(table, key, filt, M):
    """Plan tuple for M from the nearest M-bin (log distance, ties to the
    smaller bin) whose group width still fits M; None if the table has
    nothing usable.  The library's hmsv_default_plan makes the same choice
    from its compiled-in copy of the table."""
    ent = table.get(key, {}).get(filt)
    if not ent:
        return None
    bins = sorted(int(k) for k in ent)
    for b in sorted(bins, key=lambda b: abs(math.log(b) - math.log(M))):
        G, _, wpb, blocks = ent[str(b)]
        Q = q_for(G, M)
        if Q <= QMAX[G] and lds_bytes(G, Q) <= LDS_LIMIT:
            return (G, Q, wpb, blocks)
    return None


DEVICE_KEY = "gfx950:256cu"       # MI355X: the entry compiled into the library
HEADER = os.path.join(HERE, "csrc", "tuned_plans.inc")


def emit_header(table=None, key=DEVICE_KEY) -> str:
    """C table of the tuned plans for ``key``: {is_msv, M-bin, G, waves per
    block}, read by hmsv_default_plan; then those of ``key:batch`` (plans of at
    most 32 registers per lane), is_msv + 2."""
    table = load_table() if table is None else table
    rows = []
    for sub, add in ((key, 0), (key + ":batch", 2)):
        for filt in ("msv", "ssv"):
            for b, (G, _Q, wpb, blocks) in sorted(((int(k), v) for k, v in
                                                   table.get(sub, {}).get(filt, {}).items())):
                if blocks != 0:
                    raise ValueError("tuned plans use persistent grids (blocks = 0)")
                rows.append(f"    {{{add + (1 if filt == 'msv' else 0)}, {b}, {G}, {wpb}}},")
    return ("// Tuned launch plans for " + key + " (MI355X), generated from tuned_plans.json\n"
            "// by paper_1707_09683_amd/autotune.py emit_header(); regenerated by the build.\n"
            "// {is_msv (+ 2: for batches), M-bin, G, waves per block}; Q follows from G and M.\n"
            + "\n".join(rows) + "\n")


def write_header(path=HEADER) -> str:
    text = emit_header()
    old = open(path).read() if os.path.exists(path) else None
    if old != text:
        with open(path, "w") as fh:
            fh.write(text)
    return path


def tune(nseq=500_000, bins=M_BINS, filters=("msv", "ssv"), reps=4, seed=2, log=print, qmax=64):
    import torch
    import synth
    from . import Profile, Database, msv_score, ssv_score, new_workspace, make_plan

    dev = torch.device("cuda:0")
    st = synth.streams(seed)
    db_np, _ = synth.lognormal_db(seed, nseq, None, 0.0, st)
    db = Database(db_np.res, db_np.offsets, dev)
    ws = new_workspace(dev, db.nseq)
    out = {}
    for filt in filters:
        fn = msv_score if filt == "msv" else ssv_score
        sdt = torch.uint8 if filt == "msv" else torch.int8
        s = torch.empty(db.nseq, dtype=sdt, device=dev)
        f = torch.empty(db.nseq, dtype=torch.uint8, device=dev)
        res = {}
        for M in bins:
            emis = synth.sample_emissions(st["profile"], M)
            prof = Profile.from_emissions(emis, synth.BG, dev)
            ref = None
            best = None
            for cand in candidates(filt, M, qmax):
                plan = make_plan(*cand)
                fn(prof, db, s, f, ws, plan)
                torch.cuda.synchronize()
                if ref is None:
                    ref = (s.clone(), f.clone())
                elif not (torch.equal(s, ref[0]) and torch.equal(f, ref[1])):
                    raise RuntimeError(f"plan {cand} disagrees with {best} at {filt} M={M}")
                # back-to-back launches so host enqueue time stays hidden
                e0 = torch.cuda.Event(enable_timing=True)
                e1 = torch.cuda.Event(enable_timing=True)
                e0.record()
                for _ in range(reps):
                    fn(prof, db, s, f, ws, plan)
                e1.record()
                torch.cuda.synchronize()
                t = e0.elapsed_time(e1) / reps
                if best is None or t < best[0]:
                    best = (t, cand)
            gcups = M * db.residues / (best[0] * 1e-3) / 1e9
            log(f"{filt} M={M}: best {best[1]} {best[0]:.3f} ms {gcups:.0f} GCUPS", flush=True)
            res[str(M)] = list(best[1])
        out[filt] = res
    db.close()
    return out


CHOICE_DBS = ((2000, "uniform"), (3000, "lognormal"), (10_000, "lognormal"), (30_000, "lognormal"),
              (60_000, "uniform"), (100_000, "lognormal"), (167_000, "uniform"),
              (300_000, "lognormal"))
CHOICE_M = (30, 60, 100, 164, 250, 400, 600, 1000, 1500, 2400)
CHOICE_FIELDS = ("kind", "M", "nseq", "lens", "plan", "us", "best", "best_us")


def choices(path, kinds=("ssv", "p7"), log=print):
    """Times of the plans that SSV and P7Viterbi calls choose, and of the fastest."""
    import csv

    import numpy as np
    import torch
    import synth
    import paper_1707_09683_amd as hm

    def timed(fn):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        fn()
        reps, best = 1, None
        for _ in range(4):
            a.record()
            for _ in range(reps):
                fn()
            b.record()
            torch.cuda.synchronize()
            us = a.elapsed_time(b) * 1e3 / reps
            best = us if best is None else min(best, us)
            reps = max(1, min(50, int(4000 / us)))
        return best

    out = []
    for nseq, lens in CHOICE_DBS:
        rng = np.random.default_rng(nseq)
        L = synth.sample_lengths_uniform(rng, nseq, 50, 500) if lens == "uniform" else \
            synth.sample_lengths_lognormal(rng, nseq)
        res, off = synth.sample_residues(rng, L)
        db = hm.Database(res, off)
        ws = hm.new_workspace("cuda", nseq)
        for kind in kinds:
            dt = torch.int8 if kind == "ssv" else torch.int16
            s = torch.empty(nseq, dtype=dt, device="cuda")
            f = torch.empty(nseq, dtype=torch.uint8, device="cuda")
            for M in CHOICE_M:
                if M * nseq > (2 * 10 ** 8 if kind == "ssv" else 4 * 10 ** 7):
                    continue
                emis = synth.sample_emissions(rng, M)
                if kind == "ssv":
                    prof = hm.Profile.from_emissions(emis, synth.BG)
                    cand = [c[:3] for c in candidates("ssv", M) if c[2] in (4, 8, 12)]
                    chosen = hm.db_default_plan(db, "ssv", M).as_tuple()[:3]
                else:
                    prof = hm.P7Profile.from_probabilities(emis, synth.sample_transitions(rng, M),
                                                           synth.BG)
                    cand = [(G, q_for(G, M), w) for G in (4, 8, 16, 32, 64) for w in (4, 8, 16)
                            if q_for(G, M) <= (22 if G == 64 else 16) and (w <= 8 or G == 64)]
                    chosen = None
                call = hm.ssv_score if kind == "ssv" else hm.p7_score
                us = timed(lambda: call(prof, db, s, f, workspace=ws))
                best = None
                for c in cand:
                    plan = hm.make_plan(*c)
                    try:
                        t = timed(lambda: call(prof, db, s, f, workspace=ws, plan=plan))
                    except hm.HmsvError:
                        continue          # not built for blocks of this size
                    if best is None or t < best[0]:
                        best = (t, c)
                row = (kind, M, nseq, lens, ":".join(map(str, chosen)) if chosen else "",
                       round(us, 1), ":".join(map(str, best[1])), round(best[0], 1))
                out.append(row)
                log(*row, flush=True)
        db.close()
    with open(path, "w", newline="") as fh:
        w = csv.writer(fh)
        w.writerow(CHOICE_FIELDS)
        w.writerows(out)
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--nseq", type=int, default=500_000)
    ap.add_argument("--reps", type=int, default=4)
    ap.add_argument("--out", default=TABLE)
    ap.add_argument("--filters", default="msv,ssv",
                    help="comma-separated filters to tune; the others keep their entries")
    ap.add_argument("--bins", default="",
                    help="comma-separated M-bins to tune (default: all); the others keep "
                         "their entries")
    ap.add_argument("--emit-header", action="store_true",
                    help="only write csrc/tuned_plans.inc from tuned_plans.json")
    ap.add_argument("--batch", action="store_true",
                    help="tune the plans that queries of a batch start from (at most 32 "
                         "registers per lane)")
    ap.add_argument("--choices", default="", metavar="FILE",
                    help="time the plans that calls choose against all others instead")
    a = ap.parse_args()
    if a.choices:
        sys.path.insert(0, os.path.dirname(HERE))
        choices(a.choices)
        return
    if a.emit_header:
        print(write_header())
        return
    sys.path.insert(0, os.path.dirname(HERE))
    t0 = time.time()
    bins = tuple(int(b) for b in a.bins.split(",")) if a.bins else M_BINS
    res = tune(a.nseq, bins=bins, reps=a.reps, filters=tuple(a.filters.split(",")),
               qmax=32 if a.batch else 64)
    table = load_table() if os.path.exists(a.out) else {}
    key = device_key() + (":batch" if a.batch else "")
    dev = table.setdefault(key, {})
    for filt, ent in res.items():
        dev.setdefault(filt, {}).update(ent)
    table.setdefault("_meta", {})[key] = {
        "nseq": a.nseq, "seconds": round(time.time() - t0, 1),
        "note": "fastest plan per (filter, M-bin) on a lognormal database sample"}
    with open(a.out, "w") as fh:
        json.dump(table, fh, indent=1, sort_keys=True)
    print("wrote", a.out)


if __name__ == "__main__":
    main()
