"""The cost form of the P7Viterbi recurrence (csrc/p7_fast.hpp) against the
oracle, on the CPU: a model of the kernel's arithmetic (costs, u16 cells with
a floor at 0, the frame, I~ and D~, J opened by c, the delete chains only
where they matter) over random tables from the whole range the form accepts.
A sequence the model gives up must be one the kernel leaves to the general
kernel; every other one must equal the oracle."""
import numpy as np
import pytest

import oracle
from oracle import p7 as op7

BIAS, MAXTBM, MAXDM, DEAD = 1024, 4000, 1900, -20000
BASE = 2048 + 16 * (BIAS + 64)
NEG, POS = -32768, 32767


def tables(rng, M, kind):
    """Tables with every transition <= 0, emissions <= BIAS."""
    msc = np.full((32, M), NEG, np.int64)
    if kind == "wide":
        msc[:27] = rng.integers(-3000, BIAS + 1, size=(27, M))
        tr = -rng.integers(0, 1500, size=(7, M))
        tr[5] = -rng.integers(0, MAXDM + 1, size=M)
    else:
        msc[:27] = np.where(rng.random((27, M)) < 0.08, rng.integers(60, 220, (27, M)),
                            -rng.integers(0, 200, (27, M)))
        tr = -rng.integers(0, 160, size=(7, M))
        tr[5] = -rng.integers(0, 200, size=M)
    msc[20] = NEG
    if kind == "holes":
        msc[:20][rng.random((20, M)) < 0.05] = NEG
        tr[rng.random((7, M)) < 0.1] = NEG
        # a node that D cannot leave to M has no D->D either
        tr[6][tr[5] == NEG] = NEG
    tr[:, M - 1] = NEG
    tbm = int(-rng.integers(0, MAXTBM + 1)) if kind == "wide" else \
        int(op7.q(2.0 / (M * (M + 1.0))))
    return {"M": M, "msc": msc.astype(np.int16), "trans": tr.astype(np.int16), "tbm": tbm}


def model(prof, x, G, Q):
    """(score, flag) or None (left to the general kernel), lazily completed
    delete chains over 2G elements of Q slots."""
    M = prof["M"]
    msc, tr = prof["msc"].astype(np.int64), prof["trans"].astype(np.int64)
    mm, mi, md, im, ii, dm, dd = tr
    n = 2 * G * Q
    NONE = 65535
    cost = lambda s, add=0: np.clip(add - s, 0, NONE)
    ecost = np.full((32, n), NONE)
    ecost[:, 1:M + 1] = cost(msc, BIAS)
    ecost[20] = NONE
    cMM, cMI, cII, cMD = (np.full(n, NONE) for _ in range(4))
    sDD = np.full(n, NEG)
    cMI[1:M + 1] = cost(mi + im, BIAS)
    cII[1:M + 1] = cost(ii, BIAS)
    rises = []
    for s in range(2, M + 1):
        cMM[s] = cost(mm[s - 2])
        if dm[s - 1] >= -MAXDM:
            cMD[s] = cost(md[s - 2] + dm[s - 1])
            if dd[s - 2] > DEAD and dm[s - 2] >= -MAXDM:
                sDD[s] = dd[s - 2] + dm[s - 1] - dm[s - 2]
    rise = run = 0
    for s in range(2, M + 1):
        run = 0 if sDD[s] == NEG else max(0, run + sDD[s])
        rise = max(rise, run)
    L = len(x)
    lm = op7.length_model(L)
    loop, move = lm["NN"], lm["NB"]
    if L == 0:
        return max(NEG, min(POS, NEG + move)), 0
    if -loop > int((-ii).min()):
        return None
    K = 32 - move - prof["tbm"]
    F, lvl, c, fbase, ovf = BASE, BASE + K, 0, move + prof["tbm"], False
    Mv, D, I = np.zeros(n, np.int64), np.zeros(n, np.int64), np.full(n, BASE)
    sub = lambda a, b: np.maximum(a - b, 0)
    shift = lambda a: np.concatenate([[0], a[:-1]])
    for i in range(L):
        if i % 16 == 0:
            up = BASE - F
            Mv, I, D = sub(Mv + up, 0), sub(I + up, 0), sub(D + up, 0)
            c, lvl, F = max(c + up, 0), lvl + up, BASE
            fbase += (16 * BIAS if i else 0) - up
        assert max(Mv.max(), I.max(), D.max(), c, lvl) < 0x7c00 and F >= 2048
        c, lvl = max(c - (BIAS - loop), 0), lvl - (BIAS - loop)
        F = lvl - K
        nI = np.maximum(np.maximum(sub(Mv, cMI), sub(I, cII)), F)
        Mv = sub(np.maximum(np.maximum(sub(shift(Mv), cMM), shift(I)), shift(D)), ecost[x[i]])
        I = nI
        c = max(c, int(Mv.max()))
        if c > lvl:
            lvl = c
            F = lvl - K
            I = np.maximum(I, F)
            ovf = ovf or c - BASE + fbase + (i % 16 + 1) * BIAS >= POS
        inn = sub(shift(Mv), cMD)
        D = np.zeros(n, np.int64)
        for s in range(n):
            if s % Q == 0:
                D[s] = max(inn[s], F - rise)
            else:
                D[s] = max(inn[s], D[s - 1] + sDD[s])
        while True:
            first = np.arange(0, n, Q)
            in0 = shift(D)[first] + sDD[first]
            if not (in0 > D[first]).any():
                break
            D[first] = np.maximum(D[first], in0)
            for q in range(1, Q):
                D[first + q] = np.maximum(D[first + q], D[first + q - 1] + sDD[first + q])
    if c + 1023 < F:
        return None
    C = c - BASE + fbase + ((L - 1) % 16 + 1) * BIAS - 32
    return (POS, 1) if ovf else (max(NEG, min(POS, C + move)), 0)


@pytest.mark.parametrize("kind", ["usual", "holes", "wide"])
def test_cost_form_equals_oracle(kind):
    rng = np.random.default_rng({"usual": 1, "holes": 2, "wide": 3}[kind])
    scored = left = over = 0
    for trial in range(40):
        M = int(rng.integers(1, 40))
        G = int(rng.choice([1, 2, 4]))
        Q = -(-(M + 1) // (2 * G)) + int(rng.integers(0, 2))
        prof = tables(rng, M, kind)
        best = prof["msc"][:20].argmax(0)
        for _ in range(6):
            L = int(rng.integers(0, 120))
            x = rng.integers(0, 27, size=L).astype(np.uint8)
            if rng.random() < 0.6 and L:             # runs of the best residues: J opens
                x = np.resize(best, L).astype(np.uint8)
                hit = rng.random(L) < 0.05
                x[hit] = rng.integers(0, 27, size=int(hit.sum()))
            got = model(prof, x, G, Q)
            if got is None:
                left += 1
                continue
            exp = oracle.p7_seq(prof, x)
            assert got == exp, (kind, trial, M, G, Q, L, got, exp)
            scored += 1
            over += exp[1]
    assert scored > 100 and (kind != "wide" or over > 5), (scored, left, over)
