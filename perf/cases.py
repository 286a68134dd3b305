"""The calls whose speed is measured: searches a user of this package runs.

A search scores one profile HMM against a protein database that is already
packed in device memory: the MSV or SSV filter, the gapped P7Viterbi filter,
the three-stage pipeline, a batch of profiles in one graph launch, or one
range of the database.  Profile lengths lie in Pfam's range and the lengths
of the sequences are log-normal (mean about 350 residues) unless the case
says otherwise.  A case is a dict of plain values:

  name    only the listed ones
  kind    "msv", "ssv", "p7", "pipeline", "batch" or "range"
  M       nodes of the profile (batch: of the longest profile)
  nseq    sequences of the database
  lens    "lognormal" or "uniform" (50..500 residues)
  degen   share of the residues that are degenerate codes (B, J, Z, U, O, X)
  queries profiles of a batch (1 elsewhere)
  plain   True: the call is given nothing but the profile and the database;
          False: the program keeps outputs and workspace and passes them
"""
import math

import numpy as np
import torch

import paper_1707_09683_amd as hm
from paper_1707_09683_amd.batch import Batch

# Amino-acid background in thousandths (sums to 1000), in code order
# ACDEFGHIKLMNPQRSTVWY.
_BG1000 = (74, 25, 54, 54, 47, 74, 26, 68, 58, 99, 25, 45, 39, 34, 52, 57, 51, 73, 13, 32)
BG = np.array(_BG1000, dtype=np.float64) / 1000.0
_MU, _SIGMA, _LMIN, _LMAX = 5.5825, 0.7422, 20, 35000
_MEAN = {"lognormal": math.exp(_MU + _SIGMA * _SIGMA / 2), "uniform": 275.0}
_PASS = 0.022             # share of the sequences the filter stage passes on to P7Viterbi


def _case(kind, M, nseq, lens="lognormal", degen=0.0, queries=1, plain=False, name=None):
    c = {"kind": kind, "M": M, "nseq": nseq, "lens": lens, "degen": degen, "queries": queries,
         "plain": plain}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one short profile against a small set, as in a script or a test:
        # the call with nothing kept between searches
        _case("msv", 48, 2000, "uniform", plain=True, name="msv_m48_2k"),
        # a proteome-sized set and an ordinary domain profile
        _case("ssv", 151, 20011, name="ssv_m151_20k"),
        # the shortest families against a large database
        _case("msv", 30, 500_000, name="msv_m30_500k"),
        # short domain profiles, the first filter stage
        _case("ssv", 100, 200_000, name="ssv_m100_200k"),
        # the headline search
        _case("msv", 400, 500_000, name="msv_m400_500k"),
        # long profiles
        _case("ssv", 1000, 100_000, name="ssv_m1000_100k"),
        _case("msv", 2400, 60_000, name="msv_m2400_60k"),
        # real databases carry ambiguous residues: 27-row score tables, odd sizes
        _case("msv", 187, 50_021, degen=0.02, name="msv_m187_degenerate"),
        # the gapped filter over a whole database, short and ordinary profiles
        _case("p7", 100, 200_000, name="p7_m100_200k"),
        _case("p7", 400, 200_000, name="p7_m400_200k"),
        # the three stages of a search, 2.2% of the sequences reaching P7Viterbi
        _case("pipeline", 400, 500_000, name="pipeline_m400_500k"),
        # several queries of mixed length against one database, one graph launch
        _case("batch", 1800, 60_000, queries=8, name="batch_8q_60k"),
    ]


def draw(rng):
    top = max(work(c)["flops"] for c in listed())

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["msv", "ssv", "msv", "ssv", "p7", "p7", "pipeline", "batch", "range"])
        nseq = log_int(2000, 500_000)
        M = log_int(30, 2400)
        c = _case(kind, M, nseq, rng.choice(["lognormal", "lognormal", "lognormal", "uniform"]),
                  rng.choice([0.0, 0.0, 0.0, 0.02]),
                  rng.randrange(2, 9) if kind == "batch" else 1,
                  kind in ("msv", "ssv", "p7") and rng.random() < 0.25)
        if c["degen"] and M > (2047 if kind in ("p7", "pipeline") else 2559):
            continue
        if work(c)["flops"] <= top:
            return c


# ---- inputs ------------------------------------------------------------------


def _emissions(rng, M):
    """Dirichlet(0.5 background) per node, drawn in log space."""
    a = 0.5 * BG
    g = np.log(rng.gamma(a + 1.0, size=(M, 20)))
    g += np.log(np.maximum(rng.random((M, 20)), np.finfo(np.float64).tiny)) / a
    g -= g.max(axis=1, keepdims=True)
    e = np.exp(g)
    return e / e.sum(axis=1, keepdims=True)


def _transitions(rng, M):
    """Dirichlet transitions: matches dominate, gaps are rare and short."""
    t = np.empty((M, 7))
    t[:, 0:3] = rng.dirichlet(20.0 * np.array([0.90, 0.05, 0.05]), size=M)
    t[:, 3:5] = rng.dirichlet(20.0 * np.array([0.60, 0.40]), size=M)
    t[:, 5:7] = rng.dirichlet(20.0 * np.array([0.70, 0.30]), size=M)
    return t


def _residues(case, seed, emissions):
    """Residue codes and offsets (host arrays): i.i.d. from the background,
    1% of the sequences with a segment that one of the profiles emits."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    n = case["nseq"]
    if case["lens"] == "uniform":
        L = torch.randint(50, 501, (n,), generator=g, device=dev)
    else:
        z = torch.randn(n, generator=g, device=dev, dtype=torch.float64)
        L = torch.exp(z * _SIGMA + _MU).round().clamp(_LMIN, _LMAX).to(torch.int64)
    off = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    torch.cumsum(L, 0, out=off[1:])
    total = int(off[-1])
    table = torch.repeat_interleave(torch.arange(20, dtype=torch.uint8),
                                    torch.tensor(_BG1000)).to(dev)
    res = torch.empty(total, dtype=torch.uint8, device=dev)
    for a in range(0, total, 1 << 26):
        b = min(total, a + (1 << 26))
        res[a:b] = table[torch.randint(0, 1000, (b - a,), generator=g, device=dev,
                                       dtype=torch.int32)]
    ids = torch.randperm(n, generator=g, device=dev)[:n // 100]
    which = torch.randint(0, len(emissions), (ids.numel(),), generator=g, device=dev)
    for p, e in enumerate(emissions):
        i = ids[which == p]
        if not i.numel():
            continue
        cdf = torch.from_numpy(np.cumsum(e, axis=1)).to(dev)
        M = e.shape[0]

        def uniform(hi):                     # 0 .. hi inclusive, per sequence
            u = torch.rand(i.numel(), generator=g, device=dev, dtype=torch.float64)
            return torch.minimum((u * (hi + 1)).to(torch.int64), hi)

        most = torch.clamp(L[i], max=M)
        ln = (most + 1) // 2 + uniform(most - (most + 1) // 2)
        k0, at = uniform(M - ln), off[i] + uniform(L[i] - ln)
        step = torch.arange(int(ln.sum()), device=dev)
        step -= torch.repeat_interleave(torch.cumsum(ln, 0) - ln, ln)
        rows = cdf[torch.repeat_interleave(k0, ln) + step]
        u = torch.rand(rows.shape[0], 1, generator=g, device=dev, dtype=torch.float64)
        code = (rows < u * rows[:, -1:]).sum(1).clamp(max=19).to(torch.uint8)
        res[torch.repeat_interleave(at, ln) + step] = code
    if case["degen"]:
        k = max(1, int(case["degen"] * total))
        at = torch.randint(0, total, (k,), generator=g, device=dev)
        res[at] = (21 + at % 6).to(torch.uint8)
    return res.cpu().numpy(), off.cpu().numpy()


def _lengths_of(case, rng):
    """Profile lengths of a batch: the longest, the rest spread below it."""
    M, q = case["M"], case["queries"]
    low = min(30, M)
    return [M] + [int(round(math.exp(rng.uniform(math.log(low), math.log(M)))))
                  for _ in range(q - 1)]


def _inputs(case, seed):
    rng = np.random.default_rng(seed)
    Ms = [case["M"]]
    if case["kind"] == "batch":
        # the lengths belong to the case, the profiles to the seed
        Ms = _lengths_of(case, np.random.default_rng(case["M"] * 64 + case["queries"]))
    emis = [_emissions(rng, m) for m in Ms]
    trans = _transitions(rng, Ms[0]) if case["kind"] in ("p7", "pipeline") else None
    res, off = _residues(case, seed, emis)
    return emis, trans, res, off


def prepare(case, seed):
    emis, trans, res, off = _inputs(case, seed)
    dev = torch.device("cuda", torch.cuda.current_device())
    kind, n = case["kind"], case["nseq"]
    db = hm.Database(res, off, dev)
    s = {"case": case, "db": db}
    if kind == "batch":
        profs = [hm.Profile.from_emissions(e, BG, dev) for e in emis]
        s["batch"] = Batch([("msv" if i % 2 == 0 else "ssv", p) for i, p in enumerate(profs)],
                           db, branches=4)
        s["profiles"] = profs
        return s
    if kind in ("p7", "pipeline"):
        s["p7"] = hm.P7Profile.from_probabilities(emis[0], trans, BG, dev)
    if kind != "p7":
        s["prof"] = hm.Profile.from_emissions(emis[0], BG, dev)
    if case["plain"]:
        return s
    s["ws"] = hm.new_workspace(dev, n)
    if kind == "pipeline":
        # the threshold a user calibrates: the score that about 2.2% reach
        score, _ = hm.msv_score(s["prof"], db, workspace=s["ws"])
        kth = max(1, int(n * _PASS))
        s["threshold"] = int(torch.sort(score.to(torch.int32), descending=True)[0][kth - 1])
        return s
    s["score"] = torch.zeros(n, dtype={"msv": torch.uint8, "p7": torch.int16}.get(kind, torch.int8),
                             device=dev)
    s["flags"] = torch.zeros(n, dtype=torch.uint8, device=dev)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        s["batch"].launch()
        return s["batch"].scores, s["batch"].flags
    if kind == "pipeline":
        r = hm.pipeline("msv", s["prof"], s["p7"], s["db"], s["threshold"], workspace=s["ws"])
        # the survivors' positions fill the front of their buffer
        return r.filter_score, r.filter_flags, r.count, r.p7_score, r.p7_flags
    if kind == "range":
        first, count = _range_of(case)
        return hm.score_range("ssv", s["prof"], s["db"], first, count, s["score"], s["flags"],
                              workspace=s["ws"])
    fn = {"msv": hm.msv_score, "ssv": hm.ssv_score, "p7": hm.p7_score}[kind]
    prof = s["p7"] if kind == "p7" else s["prof"]
    if case["plain"]:
        return fn(prof, s["db"])
    return fn(prof, s["db"], s["score"], s["flags"], workspace=s["ws"])


def _range_of(case):
    """A chunk as the search server issues it: from a quarter of the
    processing order (longest first), half of the sequences."""
    return case["nseq"] // 4, case["nseq"] // 2


# ---- the work of one pass ------------------------------------------------------


def work(case):
    """bytes: residues, one 16-byte record per sequence and the outputs;
    flops: per cell two operations of the MSV and SSV filters (the
    saturating add of the score and the maximum), fourteen of P7Viterbi
    (eight saturating adds and six maxima, Plan-7 recurrence)."""
    n, res = case["nseq"], case["nseq"] * _MEAN[case["lens"]]
    kind = case["kind"]
    if kind == "range":
        # the middle half of the length order holds about this share
        n, res = n / 2, res * (0.38 if case["lens"] == "lognormal" else 0.5)
    Ms = [case["M"]]
    if kind == "batch":
        Ms = _lengths_of(case, np.random.default_rng(case["M"] * 64 + case["queries"]))
    per_cell = 14.0 if kind == "p7" else 2.0
    flops = per_cell * sum(Ms) * res
    nbytes = len(Ms) * (res + (19.0 if kind == "p7" else 18.0) * n)
    if kind == "pipeline":
        flops += 14.0 * case["M"] * res * _PASS
        nbytes += _PASS * (res + 19.0 * n) + 8.0 * n
    return {"bytes": nbytes, "flops": flops}


# ---- the filters in plain integers ---------------------------------------------


def _tables(emis):
    """Third-bit scores r[x, k] (x < 27; -inf as -10**6) and dbias."""
    def rhaz(v):
        return np.sign(v) * np.floor(np.abs(v) + 0.5)

    neg = -10 ** 6
    with np.errstate(divide="ignore"):
        lg = np.log2(emis / BG)
    r = np.full((32, emis.shape[0]), neg, dtype=np.int64)
    r[:20] = np.where(np.isfinite(lg), rhaz(3.0 * lg), neg).T.astype(np.int64)
    dbias = int(r[:20].max())
    groups = {21: (2, 11), 22: (7, 9), 23: (3, 13), 24: (1,), 25: (8,), 26: tuple(range(20))}
    for code, members in groups.items():
        num = np.zeros(emis.shape[0])
        den = 0.0
        for x in members:
            num, den = num + BG[x] * lg[:, x], den + BG[x]
        m = num / den
        r[code] = np.where(np.isfinite(m), rhaz(3.0 * m), neg).astype(np.int64)
    return r, dbias


def _cost(p):
    v = 3.0 * math.log2(p)
    return int(-math.copysign(math.floor(abs(v) + 0.5), v))


def exact(case, seed):
    """Scores and flags of the MSV or SSV filter by the definition: one row at
    a time over all sequences still running.  None for the other kinds (the
    delete chain of P7Viterbi runs node by node) and for large cases."""
    if case["kind"] not in ("msv", "ssv") or work(case)["flops"] > 2e10:
        return None
    emis, _, res, off = _inputs(case, seed)
    r, dbias = _tables(emis[0])
    M, n, dev = case["M"], case["nseq"], torch.device("cuda")
    cost = torch.from_numpy(np.minimum(255, dbias - r)).to(dev)
    sc = torch.clamp(dbias - cost, min=-128)
    L = torch.from_numpy(np.diff(off)).to(dev)
    order = torch.argsort(L, descending=True)
    start, Ls = torch.from_numpy(off[:-1]).to(dev)[order], L[order]
    text = torch.from_numpy(res).to(dev)
    live = torch.searchsorted(-Ls, -torch.arange(int(Ls[0]) if n else 0, device=dev),
                              side="left").tolist()      # sequences longer than i
    msv = case["kind"] == "msv"
    lo = 0 if msv else -128
    cells = torch.full((n, M + 1), lo, dtype=torch.int64, device=dev)
    over = torch.zeros(n, dtype=torch.bool, device=dev)
    best = torch.full((n,), lo, dtype=torch.int64, device=dev)
    if msv:
        tbm = _cost(2.0 / (M * (M + 1.0)))
        uniq, inv = torch.unique(Ls, return_inverse=True)
        tjb = torch.tensor([_cost(3.0 / (l + 3.0)) for l in uniq.tolist()], device=dev)[inv] + tbm
        scb = torch.clamp(190 - tjb, min=0)
    for i, m in enumerate(live):
        x = text[start[:m] + i].to(torch.int64)
        prev = cells[:m, :-1]
        if msv:
            v = torch.clamp(torch.maximum(prev, scb[:m, None]) + dbias, max=255) - cost[x]
            v = torch.clamp(v, min=0)
            top = v.max(1)[0]
            over[:m] |= top >= 255 - dbias
            best[:m] = torch.maximum(best[:m], torch.clamp(top - 3, min=0))
            scb[:m] = torch.clamp(torch.clamp(best[:m], min=190) - tjb[:m], min=0)
        else:
            v = torch.clamp(prev + sc[x], -128, 127)
            best[:m] = torch.maximum(best[:m], v.max(1)[0])
        cells[:m, 1:] = v
    if not msv:
        over = best == 127
    best[over] = 255 if msv else 127
    score = torch.empty(n, dtype=torch.uint8 if msv else torch.int8, device=dev)
    flags = torch.empty(n, dtype=torch.uint8, device=dev)
    score[order], flags[order] = best.to(score.dtype), over.to(torch.uint8)
    return score, flags
