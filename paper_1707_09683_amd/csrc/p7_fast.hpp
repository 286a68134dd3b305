// P7Viterbi, the kernel that scores almost every sequence: the recurrence of
// p7_kernel.hpp with 9.5 instead of 14 packed instructions per cell pair.
//
// What bounds the kernel is VALU issue, so the recurrence is rewritten for
// fewer instructions; every rewrite is exact for the values that can reach a
// score, and the few sequences (and the profiles) it is not proven for go to
// p7_kernel.
//
//  * Frame.  Cells hold u = v - frame in 0..31743, v the score.  The frame
//    rises by kP7Bias per row, so every emission and transition is a cost
//    >= 0 and one unsigned saturating subtract (v_pk_sub_u16 clamp, floor 0);
//    at each 16-row step it is moved so that the floor F below sits at kP7Base.
//    u stays below 31744, so its bit pattern read as fp16 orders like the
//    integer and v_pk_maximum3_f16 takes three values at once.
//  * Floor.  Every M of row i + 1 is at least F - cost(e), F = B + tBM of row
//    i.  With no transition score above 0, a value below F can reach no cell
//    but through a term below F: it changes no score.  F >= 2048 in
//    the frame, so the floor at 0 only touches such values.  (F falls by the
//    length model's loop score per row, and rises where J opens.)
//  * I~ = I + tIM of its node: M takes it without an add.  I~ also holds F
//    (max3), so M needs no separate B term; F passed on through I~ stays at
//    or below the next row's F if no I->I cost is below |loop|.
//  * D~ = D + tDM of its node, its D->D cost corrected by the difference of
//    the two nodes' tDM (it can be negative: a signed add).
//  * E and C: c is the running max of E, decayed by loop per row (C + 32),
//    kept per lane.  J (= C) matters only once it passes N: a lane whose c
//    passes lvl = max(N, J) + 32 makes the group take its maximum and raise
//    lvl and F.  No reduction across lanes otherwise.
//  * The M, D shifted across lanes for the D pass serve the next row.
//
// Per pair of cells: M sub, max3, sub; I~ sub, sub, max3; D~ sub, add, max;
// c half a max3.  200,000 lognormal sequences, p7_kernel alone and with this
// kernel before it: M = 400 (16 lanes x 13) 8.45 -> 6.19 ms, 234 -> 167 VALU
// instructions per wavefront row (160 since delete chains end at their own
// slot's bound); M = 100 (8 x 7) 5.13 -> 3.75 ms, 146 -> 103 (102; half of that
// call is the tail of its longest records).  A last chunk of one register (Q = 13)
// is read as 4 bytes of its 16, in four passes of the LDS: six such reads a row,
// 15.7 bank conflict cycles.
//
// Conditions on the profile (by the prep kernel): transitions <= 0,
// emissions <= kP7Bias, tBM in [-kP7MaxTbm, 0], and D->M of every node at
// least -kP7MaxDm unless its D->D is -inf too.  Not so: p7_kernel runs every
// record.  Per sequence: |loop| at most the smallest I->I cost, which holds
// down to some length: this kernel lists the shorter ones for p7_kernel
// as it starts.  And C no more than 1023 below F at the end; else its
// position joins that list (sequences of non-scoring residues).  (Each short
// one a step here and an atomic for its place in the list: 100,000 sequences of
// 10 to 60 residues on a profile with an I->I cost of 0, M = 100 1371 us; now
// 189.)
#pragma once
#include <algorithm>
#include "p7_kernel.hpp"

namespace hmsv {

__device__ __forceinline__ uint32_t usub(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, a),
                                                                      __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t uadd(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, a) + __builtin_bit_cast(u16x2, b));
}
__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t imax2(uint32_t a, uint32_t b) {
    return s16_bits(smax(as_s16x2(a), as_s16x2(b)));
}
__device__ __forceinline__ uint32_t iadd(uint32_t a, uint32_t b) {
    return s16_bits(adds(as_s16x2(a), as_s16x2(b)));
}
__device__ __forceinline__ uint32_t splat_u(int v) {
    return (uint32_t)(v & 0xffff) * 0x10001u;
}

// Registers of transition costs per lane: a lane with at most this many
// registers per state keeps the five transition rows in VGPRs and reads each
// row's emission costs one row ahead (wide groups run the longest records,
// alone on their SIMD at the end of a call: latency bounds them).
constexpr int kP7RegQ = 6;

template <int G, int Q, int THREADS>
__global__ void __launch_bounds__(THREADS) p7_fast_kernel(P7Args a) {
    using Lay = Layout<G, Q, kP7Rows>;
    constexpr int RS = Lay::RS;
    constexpr int NCH = (Q + 3) / 4;
    constexpr bool REG = Q <= kP7RegQ;
    if (!p7_profile_fast(a)) return;          // p7_kernel runs every record
    // (Read before anything is stored, these stay scalars.  After, they took two
    // VGPRs, and 32 lanes x 16 registers past 128: M = 1000 on 500,000 sequences
    // 36.2 ms, now 28.5.)
    const int32_t *sel = a.sel;
    const int nseq = a.aux[kAuxFast], minii = a.aux[kAuxMinII], all = p7_records(a);
    // the records not taken here, for p7_kernel
    for (int i = nseq + (int)(blockIdx.x * blockDim.x + threadIdx.x); i < all;
         i += (int)(gridDim.x * blockDim.x))
        a.pend[i - nseq] = sel ? sel[i] : i;
    extern __shared__ uint32_t lds[];
    {
        const uint4 *src = (const uint4 *)a.fimage;
        uint4 *dst = (uint4 *)lds;
        const int n16 = (a.rows + kFRows) * (RS / 4);
        for (int i = threadIdx.x; i < n16; i += blockDim.x) dst[i] = src[i];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int j = lane % G;
    const bool gstart = j == 0;
    // of the first slots of the lane's two elements
    const uint32_t rise = (uint32_t)a.rise[2 * j * Q] | ((uint32_t)a.rise[(2 * j + 1) * Q] << 16);
    const uint32_t *T[3] = {lds + Lay::lane_off(lane, 4),
                            lds + Lay::OFF2 + Lay::lane_off(lane, 2),
                            lds + Lay::OFF1 + Lay::lane_off(lane, 1)};
    // registers 4ch .. 4ch+3 of table row r
    auto load = [&](uint32_t r, auto ch_c, uint32_t (&d)[4]) {
        constexpr int ch = decltype(ch_c)::value;
        const uint32_t rb = r * (uint32_t)(RS * 4);
        if constexpr (ch < Lay::NF) {
            const uint4 v = *(const uint4 *)((const char *)T[0] + rb + ch * Lay::CW * 4);
            d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
        } else {
            if constexpr (Lay::T2) {
                const uint2 v = *(const uint2 *)((const char *)T[1] + rb);
                d[0] = v.x; d[1] = v.y;
            }
            if constexpr (Lay::T1)
                d[Lay::T2 ? 2 : 0] = *(const uint32_t *)((const char *)T[2] + rb);
        }
    };
    auto load_all = [&](uint32_t r, uint32_t (&d)[NCH * 4]) {
        [&]<int... C>(std::integer_sequence<int, C...>) {
            (([&] {
                 uint32_t t4[4] = {0u, 0u, 0u, 0u};
                 load(r, std::integral_constant<int, C>{}, t4);
#pragma unroll
                 for (int u = 0; u < 4; ++u) d[C * 4 + u] = t4[u];
             }()),
             ...);
        }(std::make_integer_sequence<int, NCH>{});
    };
    auto residue = [](uint32_t w, int r) -> uint32_t { return (w >> (8 * r)) & 0xffu; };
    const uint32_t rT = (uint32_t)a.rows;    // first transition row
    constexpr int RQ = REG ? NCH * 4 : 1;
    uint32_t tMM[RQ], tMI[RQ], tII[RQ], tMD[RQ], tDD[RQ];
    if constexpr (REG) {
        load_all(rT + kFMM, tMM);
        load_all(rT + kFMI, tMI);
        load_all(rT + kFII, tII);
        load_all(rT + kFMD, tMD);
        load_all(rT + kFDD, tDD);
    }

    // Records run longest first.  A group starts on the record of its own
    // number (see wave_rank).  Later records are claimed when
    // the current one has at most 48 rows left, in three steps of 16: the claim,
    // its value and the record's load, the last rows.  (Claimed a record or two
    // ahead, as the filter kernels do, a long record holds back what was claimed
    // behind it, and P7's rows are long enough to hide the claim.)
    const int gid = wave_rank() * (64 / G) + lane / G;
    const int ngroups = (int)(gridDim.x * (blockDim.x >> 6)) * (64 / G);
    const int nparts = (int)(gridDim.x < (unsigned)kP7Parts ? gridDim.x : (unsigned)kP7Parts);
    const int part = (int)(blockIdx.x % (unsigned)nparts);
    uint32_t *ctr = a.fqueue + part * 32;
    // claims of the wavefront's last issue: lane 0 holds the counter's value, a
    // claiming group's first lane its rank among them
    uint32_t cbase = 0u, crank = 0u;
    auto issue = [&](bool want) {
        const bool w = want && gstart;
        const unsigned long long m = __ballot(w);
        if (lane == 0) cbase = atomicAdd(ctr, (uint32_t)__popcll(m));
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (w) crank = rank;
    };
    // the claimed processing position, or -1: none left
    auto position = [&](long long r) -> int {
        if (r >= (long long)nseq) return -1;
        return sel ? sel[r] : (int)r;
    };
    auto take = [&]() -> int {
        int k = (int)crank;
        if constexpr (G > 1) k = __shfl(k, lane - j);
        k += __builtin_amdgcn_readfirstlane((int)cbase);
        return position((long long)ngroups + (long long)part + (long long)nparts * (long long)k);
    };

    uint32_t M[Q], I[Q], D[Q];
    int t = position(gid), tn = -1;
    uint4 rec = make_uint4(0u, 0u, 0u, 0u), rec16 = rec;
    uint32_t lm = 0u;
    auto load_record = [&](int p, uint4 &r, uint4 &r16, uint32_t &l) {
        if (p >= 0) {
            r = *(const uint4 *)(a.seqs + p);
            r16 = *((const uint4 *)(a.seqs + p) + 1);
            l = a.lenmodel[p];
        }
    };
    load_record(t, rec, rec16, lm);
    uint4 nrec = rec, nrec16 = rec16;
    uint32_t nlm = lm;
    int claim = 0;               // 0: none, 1: issued, 2: tn and its record loaded

    bool active = false, ovf = false, give_up = false;
    uint32_t off = a.pad_off, id = 0;
    int len = 0, done = 0;       // residues of the sequence, rows run so far
    int fbase = 0;               // score at u = kP7Base at the step's start
    int move = 0;
    // per row (packed twice): c, lvl and their common decay; K = lvl - F
    uint32_t c = 0u, lvl = 0u, delta = 0u, K = 0u, F = 0u;
    uint32_t cfin = 0u, ffin = 0u;           // c and F after the last row
    uint32_t sM = 0u, sD = 0u;               // M and D shifted one slot
    uint4 wv = make_uint4(0u, 0u, 0u, 0u);   // this step's 16 residues
    auto start = [&]() {
        active = t >= 0;
        off = active ? rec.x : a.pad_off;
        id = rec.z;
        len = active ? (int)rec.w : 0;
        done = 0;
        const int loop = active ? (int)(short)(lm & 0xffffu) : 0;
        move = active ? (int)(short)(lm >> 16) : 0;
        ovf = false;
        give_up = len > 0 && -loop > minii;
        if (give_up) len = 1;                // one step, then to the pending list
        const int k = -kP7Half - move - a.tbm;
        K = splat_u(k);
        delta = splat_u(kP7Bias - (len > 0 && !give_up ? loop : 0));
        fbase = move + a.tbm;
        F = splat_u(kP7Base);
        lvl = splat_u(kP7Base + k);
        c = cfin = 0u;
        ffin = F;
        sM = sD = 0u;
        wv = active ? rec16 : make_uint4(0x14141414u, 0x14141414u, 0x14141414u, 0x14141414u);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            M[q] = D[q] = 0u;
            I[q] = F;
        }
    };
    start();

    for (;;) {
        if (!__any(active)) break;
        bool ended = false;
        do {
            // the next record (see above)
            const bool late = active && len - done <= 48;
            if (__any(late)) {
                const bool ready = claim == 1;
                if (__any(ready)) {
                    const int p = take();
                    if (ready) {
                        tn = p;
                        load_record(tn, nrec, nrec16, nlm);
                        claim = 2;
                    }
                }
                const bool want = late && claim == 0;
                if (__any(want)) {
                    issue(want);
                    if (want) claim = 1;
                }
            }
            // residues of the next step (the database stores every sequence
            // in whole 16-residue steps plus 16 more bytes)
            const uint4 wn = *(const uint4 *)(a.res + off + 16u);
            // the frame back to F at kP7Base (never down: a new M is at most a
            // cell or F of the row before, all at most lvl, so neither lvl nor
            // F rises within a step)
            {
                const int up = kP7Base - (int)(F & 0xffffu);
                const uint32_t add = splat_u(up);
                fbase -= up;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    M[q] = uadd(M[q], add);
                    I[q] = uadd(I[q], add);
                    D[q] = uadd(D[q], add);
                }
                sM = uadd(sM, add);
                sD = uadd(sD, add);
                c = uadd(c, add);
                lvl = uadd(lvl, add);
            }
            const int last = len - done - 1;         // the sequence's last row, if in this step
            const bool ends = __any(active && last < 16);
            uint32_t ea[REG ? NCH * 4 : 1], eb[REG ? NCH * 4 : 1];
            if constexpr (REG) load_all(residue(wv.x, 0), ea);
            // one row: residue x, row r of the step; REG: its emission costs
            // in e (the next row's are read into en)
            auto row = [&](uint32_t x, uint32_t xn, int r, uint32_t (&e)[REG ? NCH * 4 : 1],
                           uint32_t (&en)[REG ? NCH * 4 : 1]) {
                if constexpr (REG) load_all(xn, en);
                // ---- M and I~, registers in descending order ---------------
                // (in place: slot q's new M reads the old M, I~ and D~ of slot
                // q - 1, not yet overwritten; its new I~ reads its own old M
                // and I~, updated first)
                c = usub(c, delta);
                lvl = usub(lvl, delta);
                F = usub(lvl, K);
                const uint32_t sI = shift_in(I[Q - 1]);
                uint32_t pend = 0u;
                bool have = false;
                [&]<int... C>(std::integer_sequence<int, C...>) {
                    (([&] {
                         constexpr int ch = NCH - 1 - C;
                         using CH = std::integral_constant<int, ch>;
                         uint32_t ve[4], vmm[4], vmi[4], vii[4];
                         if constexpr (!REG) {
                             // one chunk's loads at a time: keeps the scheduler
                             // from hoisting every chunk's loads at once
                             __builtin_amdgcn_sched_barrier(0);
                             load(x, CH{}, ve);
                             load(rT + kFMM, CH{}, vmm);
                             load(rT + kFMI, CH{}, vmi);
                             load(rT + kFII, CH{}, vii);
                         } else {
#pragma unroll
                             for (int u = 0; u < 4; ++u) {
                                 ve[u] = e[ch * 4 + u];
                                 vmm[u] = tMM[ch * 4 + u];
                                 vmi[u] = tMI[ch * 4 + u];
                                 vii[u] = tII[ch * 4 + u];
                             }
                         }
#pragma unroll
                         for (int u = 3; u >= 0; --u) {
                             const int q = ch * 4 + u;
                             if (q >= Q) continue;
                             // (pinned here: left to itself the compiler sinks
                             // the I~ update to the row's end and keeps copies
                             // of the old M)
                             uint32_t nI = hmax3(usub(M[q], vmi[u]), usub(I[q], vii[u]), F);
                             asm volatile("" : "+v"(nI));
                             const uint32_t gM = q > 0 ? M[q - 1] : sM;
                             const uint32_t gI = q > 0 ? I[q - 1] : sI;
                             const uint32_t gD = q > 0 ? D[q - 1] : sD;
                             M[q] = usub(hmax3(usub(gM, vmm[u]), gI, gD), ve[u]);
                             I[q] = nI;
                             if (have) c = hmax3(c, pend, M[q]);
                             else pend = M[q];
                             have = !have;
                         }
                     }()),
                     ...);
                }(std::make_integer_sequence<int, NCH>{});
                if (have) c = hmax(c, pend);
                // ---- J: a cell above lvl opens or raises it -----------------
                if (__any(umax(c, lvl) != lvl)) {
                    const int cg = group_max<G>(lane_max_bits(c));
                    lvl = umax(lvl, splat_u(cg));
                    F = usub(lvl, K);
#pragma unroll
                    for (int q = 0; q < Q; ++q) I[q] = umax(I[q], F);
                    if (cg - kP7Base + fbase + (r + 1) * kP7Bias >= kP7Pos) ovf = true;
                }
                // ---- D~ within each element, ascending ---------------------
                // (from the new M; slot 0 takes the previous element's last M
                // here and its last D~ below).  Values up to F - rise reach no
                // cell above F (rise: the most that a run of D~->D~ scores from
                // that slot on adds up to), so slot 0 may be raised to that.
                // (With the largest rise of the profile for all: D->D of 0.9
                // throughout, M = 60 on 20,000 sequences 3.88 ms.)
                sM = shift_in(M[Q - 1]);
                const uint32_t thr = usub(F, rise);
                uint32_t dd0 = 0u;
                [&]<int... C>(std::integer_sequence<int, C...>) {
                    (([&] {
                         constexpr int ch = C;
                         using CH = std::integral_constant<int, ch>;
                         uint32_t vmd[4], vdd[4];
                         if constexpr (!REG) {
                             load(rT + kFMD, CH{}, vmd);
                             load(rT + kFDD, CH{}, vdd);
                         } else {
#pragma unroll
                             for (int u = 0; u < 4; ++u) {
                                 vmd[u] = tMD[ch * 4 + u];
                                 vdd[u] = tDD[ch * 4 + u];
                             }
                         }
#pragma unroll
                         for (int u = 0; u < 4; ++u) {
                             const int q = ch * 4 + u;
                             if (q >= Q) continue;
                             if (q == 0) {
                                 D[0] = umax(usub(sM, vmd[0]), thr);
                                 dd0 = vdd[0];
                             } else {
                                 D[q] = imax2(usub(M[q - 1], vmd[u]), iadd(D[q - 1], vdd[u]));
                             }
                         }
                     }()),
                     ...);
                }(std::make_integer_sequence<int, NCH>{});
                // ---- D~ chains across elements, where they matter ----------
                // (the previous element's last D~ carried along the slots while
                // it raises them; a pass ends at the first chunk whose last slot
                // stays as it was)
                // (raise: the new value in place, and whether any lane's rose)
                auto raise = [](uint32_t &d, uint32_t v) -> bool {
                    const uint32_t n = imax2(d, v);
                    const bool rose = __any(n != d);
                    d = n;
                    return rose;
                };
                auto pass = [&]() -> bool {       // true: the last slot rose, too
                    bool rose = true;
                    [&]<int... C>(std::integer_sequence<int, C...>) {
                        (([&] {
                             constexpr int ch = C;
                             constexpr int hi = ch * 4 + 3 < Q ? ch * 4 + 3 : Q - 1;
                             if (!rose) return;
                             uint32_t vdd[4];
                             if constexpr (!REG) {
                                 load(rT + kFDD, std::integral_constant<int, ch>{}, vdd);
                             } else {
#pragma unroll
                                 for (int u = 0; u < 4; ++u) vdd[u] = tDD[ch * 4 + u];
                             }
#pragma unroll
                             for (int u = 0; u < 4; ++u) {
                                 const int q = ch * 4 + u;
                                 if (q == 0 || q >= hi) continue;
                                 D[q] = imax2(D[q], iadd(D[q - 1], vdd[u]));
                             }
                             if constexpr (hi > 0) rose = raise(D[hi], iadd(D[hi - 1], vdd[hi & 3]));
                         }()),
                         ...);
                    }(std::make_integer_sequence<int, NCH>{});
                    return rose;
                };
                for (;;) {
                    sD = shift_in(D[Q - 1]);
                    if (!raise(D[0], iadd(sD, dd0)) || !pass()) break;
                }
                if (ends && r == last) {
                    cfin = c;
                    ffin = F;
                }
            };
            // four residues a turn
#pragma unroll 1
            for (int r = 0; r < 16; r += 4) {
                const uint32_t w = wv.x;
                row(residue(w, 0), residue(w, 1), r, ea, eb);
                row(residue(w, 1), residue(w, 2), r + 1, eb, ea);
                row(residue(w, 2), residue(w, 3), r + 2, ea, eb);
                row(residue(w, 3), residue(wv.y, 0), r + 3, eb, ea);
                wv.x = wv.y;
                wv.y = wv.z;
                wv.z = wv.w;
                wv.w = wn.x;
            }
            fbase += 16 * kP7Bias;
            done += 16;
            // groups without a sequence stay on the padding (>= 64 bytes of
            // code 20 at pad_off)
            if (active) off += 16u;
            wv.y = wn.y;
            wv.z = wn.z;
            wv.w = wn.w;
            ended = active && done >= len;
        } while (!__any(ended));

        // ---- finished sequences: score, then the next record ---------------
        {
            const int cg = group_max<G>(lane_max_bits(cfin));
            const bool left = ended && len > 0 &&
                              (give_up || cg + 1023 < (int)(ffin & 0xffffu));
            if (__any(left)) {                       // one atomic per wavefront
                const unsigned long long m = __ballot(left && gstart);
                uint32_t at = 0u;
                if (lane == 0) at = atomicAdd((uint32_t *)a.aux + kAuxPend, (uint32_t)__popcll(m));
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) +
                     __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                               __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                if (left && gstart) a.pend[at] = t;
            }
            if (ended && gstart && !left) {
                const int rl = (len - 1) & 15;       // its last row within the step
                const int cend = len > 0 ? cg - kP7Base + fbase - 16 * kP7Bias
                                               + (rl + 1) * kP7Bias + kP7Half
                                         : kP7Neg;
                a.score[id] = ovf ? (int16_t)kP7Pos : (int16_t)sat16(cend + move);
                a.flag[id] = ovf ? 1 : 0;
            }
        }
        if (__any(ended && claim == 1)) {        // records of at most 16 rows
            const int p = take();
            if (ended && claim == 1) {
                tn = p;
                load_record(tn, nrec, nrec16, nlm);
            }
        }
        if (ended) {
            t = tn;
            rec = nrec;
            rec16 = nrec16;
            lm = nlm;
            claim = 0;
            start();
        }
    }
}

// Blocks of up to 8 wavefronts (512 threads), or 16 for 64-lane groups of at
// most 18 registers or of 20: their LDS image allows one block per CU, so 16
// wavefronts per block is the way to 4 per SIMD.  1024 threads leave 128 VGPRs:
// p7_kernel fits them (20 to 40 bytes per lane spilt at 19, 21 and 22),
// p7_fast_kernel spills 20 bytes per lane at 18 registers and 76 at 20.  It
// pays all the same where all CUs have work to the end: M = 2400 on 100,000
// sequences 13.9 ms, 17.5 with 8 wavefronts (64 x 19 17.4, not built for 16),
// M = 2200 13.2 and 17.6; not where the longest record sets it: 20,000
// sequences, 4.79 and 4.26 ms (4.22), 4.40 and 4.36.
template <int G, int Q>
constexpr int kP7MaxWaves = (G == 64 && (Q <= 18 || Q == 20)) ? 16 : 8;

template <int G, int Q, int THREADS>
hipError_t launch_p7_kernels(const P7Args &a, int wpb, P7Blocks blocks, hipStream_t s) {
    const size_t lds = p7_lds_bytes(G, Q, a.rows), flds = p7_fast_lds_bytes(G, Q, a.rows);
    hipError_t e = hipSuccess;
    if (flds > 64 * 1024)
        e = hipFuncSetAttribute((const void *)p7_fast_kernel<G, Q, THREADS>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)flds);
    if (e == hipSuccess && lds > 64 * 1024)
        e = hipFuncSetAttribute((const void *)p7_kernel<G, Q, THREADS>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((p7_fast_kernel<G, Q, THREADS>), dim3(blocks.fast), dim3(wpb * 64), flds, s,
                       a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((p7_kernel<G, Q, THREADS>), dim3(blocks.general), dim3(wpb * 64), lds, s, a);
    return hipGetLastError();
}

// The LDS images and the profile's bounds, the cost form's kernel, then
// p7_kernel on what that left (or on everything).
template <int G, int Q>
hipError_t launch_p7(const P7Args &a, int wpb, P7Blocks blocks, hipStream_t s) {
    if (a.rows != kRows && a.rows != kDegenRows) return hipErrorInvalidValue;
    const int n = (a.rows + 7) * lds_layout(G, Q, kP7Rows).RS;
    const int fn = (a.rows + kFRows) * lds_layout(G, Q, kP7Rows).RS;
    if (wpb < 1 || wpb > kP7MaxWaves<G, Q>) return hipErrorInvalidValue;
    const int nb = (n + 255) / 256, fnb = (fn + 255) / 256;
    hipLaunchKernelGGL((p7_prep_kernel<G, Q>), dim3(nb + fnb + 2 + a.rows), dim3(256), 0, s, a, nb,
                       fnb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if constexpr (kP7MaxWaves<G, Q> > 8) {
        if (wpb > 8) return launch_p7_kernels<G, Q, 1024>(a, wpb, blocks, s);
    }
    return launch_p7_kernels<G, Q, 512>(a, wpb, blocks, s);
}

template <int G, int Q, int THREADS>
P7Blocks occupancy_p7_kernel(int wpb, int rows) {
    P7Blocks nb{0, 0};
    const size_t lds = p7_lds_bytes(G, Q, rows), flds = p7_fast_lds_bytes(G, Q, rows);
    if (hipFuncSetAttribute((const void *)p7_kernel<G, Q, THREADS>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
        hipFuncSetAttribute((const void *)p7_fast_kernel<G, Q, THREADS>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)flds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb.general, p7_kernel<G, Q, THREADS>,
                                                     wpb * 64, lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb.fast, p7_fast_kernel<G, Q, THREADS>,
                                                     wpb * 64, flds) != hipSuccess)
        return P7Blocks{0, 0};
    return P7Blocks{std::min(nb.general, lds_blocks(lds)), std::min(nb.fast, lds_blocks(flds))};
}

// Resident blocks of wpb wavefronts per CU (0 on error or an unsupported
// block size).
template <int G, int Q>
P7Blocks occupancy_p7(int wpb, int rows) {
    if (wpb < 1 || wpb > kP7MaxWaves<G, Q>) return P7Blocks{0, 0};
    if constexpr (kP7MaxWaves<G, Q> > 8) {
        if (wpb > 8) return occupancy_p7_kernel<G, Q, 1024>(wpb, rows);
    }
    return occupancy_p7_kernel<G, Q, 512>(wpb, rows);
}

}  // namespace hmsv
