// P7Viterbi (gapped Plan-7 Viterbi) filter kernel for gfx950.
//
// What it computes (paper Sec. 2.1, Eq. 1, with the Plan-7 special states
// N, B, E, C, J of the DP matrix's flanks), in int16 saturating arithmetic
// with -32768 as -inf, for residues x_1..x_L and nodes j = 1..M:
//   M[i][j] = msc_j(x_i) + max(M[i-1][j-1] + tMM, I[i-1][j-1] + tIM,
//                              D[i-1][j-1] + tDM, B[i-1] + tBM)
//   I[i][j] = max(M[i-1][j] + tMI, I[i-1][j] + tII)        (insert score 0)
//   D[i][j] = max(M[i][j-1] + tMD, D[i][j-1] + tDD)
// then per row E = max_j M, J = max(J + tJJ, E + tEJ), C = max(C + tCC,
// E + tEC), N = N + tNN, B = max(N + tNB, J + tJB); score = C[L] + tCT, or
// 32767 with the overflow flag once a row's E saturates.
//
// Mapping (as the MSV/SSV kernel): a lane group of G lanes aligns one
// sequence; each lane holds Q registers of two int16 cells for each of M,
// I and D, striped (register q, element e = lane e/2, half e%2, is slot
// q + Q e; slot 0 is a dummy node whose emissions and transitions are -inf,
// so every value it holds reaches a real node only through a -inf
// transition).  Packed saturating adds (v_pk_add_i16 clamp) and maxima
// (v_pk_max_i16) update two cells per instruction.
//
// Per row: M and I in place, registers in descending order; D within each
// element in ascending order, its first slot taking the previous element's
// last M (M->D); then the D->D chains across elements are completed
// Farrar-style ("lazy F"): each element takes the last D of the element
// before it (one DPP shift) and carries it along its slots, max-ing it in,
// while some element's last D rises to a value that can still raise a
// cell of the next row (max and a saturating add of a fixed score commute,
// so every such value is the sequential chain's; values below that bound
// change no M, no E and no score).  Scores come from LDS: 21 rows of match
// emissions by residue (27 with the degenerate codes) and 7 rows of
// transitions, in the MSV image's conflict-free layout.  The special
// states, packed int16, are updated once per row from the group's maximum.
//
// Lane groups take records (longest first) from queues as they finish one;
// the next record is loaded, and the one after it claimed, while the
// current one runs.  A sequence runs exactly L rows: the rows of the last
// 16-residue step past L leave the special states untouched.
#pragma once
#include <utility>
#include "filter_kernel.hpp"

namespace hmsv {

typedef short s16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ s16x2 as_s16x2(uint32_t v) { return __builtin_bit_cast(s16x2, v); }
__device__ __forceinline__ uint32_t s16_bits(s16x2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ s16x2 adds(s16x2 a, s16x2 b) { return __builtin_elementwise_add_sat(a, b); }
__device__ __forceinline__ s16x2 smax(s16x2 a, s16x2 b) { return __builtin_elementwise_max(a, b); }
__device__ __forceinline__ s16x2 splat16(int v) { return s16x2{(short)v, (short)v}; }

constexpr int kP7Neg = -32768;
constexpr int kP7Pos = 32767;
constexpr int kP7Half = -32;          // E->J and E->C: 32 log2(1/2)
__device__ __forceinline__ int sat16(int v) { return v < kP7Neg ? kP7Neg : (v > kP7Pos ? kP7Pos : v); }

// The cost form of the recurrence (p7_fast.hpp): its frame rises by kP7Bias per
// row and holds the floor at kP7Base at each step's start.
constexpr int kP7Bias = 1024;         // largest emission score it takes (32 bits)
constexpr int kP7MaxTbm = 4000;       // tBM in [-kP7MaxTbm, 0]
constexpr int kP7MaxDm = 1900;        // D->M in [-kP7MaxDm, 0] at nodes with a D->D
constexpr int kP7Dead = -20000;       // D->D at or below: -inf
// 16 rows of bias and the steepest loop score (-64, L = 1) above 2048
constexpr int kP7Base = 2048 + 16 * (kP7Bias + 64);
// lvl = kP7Base + E->J half + move (L < 2^24: at least -717) + tBM must stay
// below the fp16 infinity pattern
static_assert(kP7Base + 32 + 720 + kP7MaxTbm < 0x7c00, "u stays a finite fp16 pattern");

// Words of a call's workspace head (P7Args::aux), written by the prep kernel.
constexpr int kAuxMaxDm = 0;      // max over nodes of D->M
constexpr int kAuxTransOk = 1;    // transitions and tBM within the cost form's bounds
constexpr int kAuxMinII = 2;      // smallest I->I cost over the nodes
constexpr int kAuxPend = 4;       // records the cost form leaves to p7_kernel
constexpr int kAuxFast = 5;       // the call's first records, which the cost form takes
constexpr int kAuxEmisOk = 8;     // per emission row: no score above kP7Bias
static_assert((kAuxEmisOk + kDegenRows) * 4 <= (int)kWsCounterBytes, "aux words fit");

// Whether the cost form holds for the call's profile (the same for every
// wavefront of the launch).
__device__ __forceinline__ bool p7_profile_fast(const P7Args &a) {
    const int lane = threadIdx.x & 63;
    bool bad = a.aux[kAuxTransOk] == 0;
    if (lane < a.rows) bad = bad || a.aux[kAuxEmisOk + lane] == 0;
    return !__any(bad);
}

// Records of the call: the whole database's, or those that a selection pass
// left in sel[0 .. *nsel) (a device count, known only here; never more than the
// database holds).
__device__ __forceinline__ int p7_records(const P7Args &a) {
    return a.sel ? min(max(*a.nsel, 0), a.nseq) : a.nseq;
}

// Record queues.  Records come from queues (counters the prep kernel
// zeroed), longest first: a lane group claims a record as it starts one, so
// a group that drew a long sequence draws fewer others.  Blocks are spread
// over up to kP7Parts queues, each on its own 128-byte line: queue p hands
// out records p, p + P, p + 2P, ... (each longest first), so one counter's
// atomics come from a fraction of the grid.  A claim is taken (its value
// broadcast from the group's first lane) only at the group's next switch, by
// when it has returned: `issue` for the groups that claim, `take` by the
// whole wavefront.
template <int G>
struct P7Queue {
    int nparts, part, lane, j;
    uint32_t *ctr;
    uint32_t craw = 0u;

    __device__ P7Queue(uint32_t *queues, int lane_, int j_) : lane(lane_), j(j_) {
        nparts = (int)(gridDim.x < (unsigned)kP7Parts ? gridDim.x : (unsigned)kP7Parts);
        part = (int)(blockIdx.x % (unsigned)nparts);
        ctr = queues + part * 32;
    }
    __device__ __forceinline__ void issue(bool want) {    // called by the whole wavefront
        // one atomic per wavefront (by lane 0) for all of its claiming
        // groups, each group's claim its rank among them
        const bool w = want && j == 0;
        const unsigned long long m = __ballot(w);
        if (m == 0ull) return;
        uint32_t base = 0u;
        if (lane == 0) base = atomicAdd(ctr, (uint32_t)__popcll(m));
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (w) craw = base + rank;
    }
    // a processing position, or -1: none left
    __device__ __forceinline__ int take(const int32_t *sel, int nseq) {
        int k = (int)craw;
        if constexpr (G > 1) k = __shfl(k, lane - j);
        const long long r = (long long)part + (long long)nparts * (long long)k;
        if (r >= (long long)nseq) return -1;
        return sel ? sel[r] : (int)r;
    }
};

// Score of table row r (emissions by residue below a.rows, transitions
// from there) at slot s (node s; slot 0 is the dummy).
__device__ __forceinline__ int p7_slot_score(const P7Args &a, int r, int s) {
    const int M = a.M;
    if (r < a.rows) {
        if (s < 1 || s > M || r == kInvalidCode) return kP7Neg;
        return a.msc[r * M + s - 1];
    }
    // transitions: MMp, IMp, DMp, MDp, DDp come from node s - 1; MI, II
    // from node s (their table rows: MM 0, MI 1, MD 2, IM 3, II 4, DM 5, DD 6)
    const int t = r - a.rows;
    const int from = (t == kP7MI || t == kP7II) ? s : s - 1;
    if (from < 1 || from > M) return kP7Neg;
    const int row = t == kP7MMp ? 0 : t == kP7IMp ? 3 : t == kP7DMp ? 5 : t == kP7MI ? 1
                  : t == kP7II ? 4 : t == kP7MDp ? 2 : 6;
    return a.trans[row * M + from - 1];
}

// Cost (u16, 65535 for none) of a score <= add.
__device__ __forceinline__ uint32_t p7_cost(int score, int add) {
    const int v = add - score;
    return (uint32_t)(v < 0 ? 0 : v > 65535 ? 65535 : v);
}

// Entry of the cost image (see p7_fast.hpp) of table row r at slot s (node s;
// slot 0 is the dummy): emission costs below a.rows, then the transition
// rows kFMM.. : M->M into s; M->I~ and I~->I~ at s; M->D~ and D~->D~ into s.
// I~ and D~ include I->M and D->M out of their node.
__device__ __forceinline__ uint32_t p7_slot_cost(const P7Args &a, int r, int s) {
    const int M = a.M;
    const bool node = s >= 1 && s <= M;
    if (r < a.rows)
        return !node || r == kInvalidCode ? 65535u : p7_cost(a.msc[r * M + s - 1], kP7Bias);
    auto tr = [&](int row, int k) -> int { return a.trans[row * M + k - 1]; };   // out of node k
    const int t = r - a.rows;
    const bool from = s >= 2 && s <= M;      // a node s - 1 leads to node s
    switch (t) {
    case kFMM: return from ? p7_cost(tr(0, s - 1), 0) : 65535u;
    case kFMI: return node ? p7_cost(tr(1, s) + tr(3, s), kP7Bias) : 65535u;
    case kFII: return node ? p7_cost(tr(4, s), kP7Bias) : 65535u;
    case kFMD: return from && tr(5, s) >= -kP7MaxDm ? p7_cost(tr(2, s - 1) + tr(5, s), 0) : 65535u;
    default: {
        // D~ of s from D~ of s - 1: a score (s16), the nodes' D->M exchanged
        if (!from || tr(6, s - 1) <= kP7Dead || tr(5, s - 1) < -kP7MaxDm || tr(5, s) < -kP7MaxDm)
            return (uint16_t)(short)kP7Neg;
        return (uint16_t)(short)(tr(6, s - 1) + tr(5, s) - tr(5, s - 1));
    }
    }
}

// Per call: the LDS images (general_rows = a.rows + 7 rows of scores, and
// a.rows + kFRows rows of the cost form, both of the lds_layout(G, Q,
// kP7Rows) shape), one dword per thread; then one block for the profile's
// transitions, one per emission row and one for the rises: what the cost form
// and its bounds need.
template <int G, int Q>
__global__ void __launch_bounds__(256) p7_prep_kernel(P7Args a, int image_blocks,
                                                      int fimage_blocks) {
    constexpr LdsLayout D = lds_layout(G, Q, kP7Rows);
    const int check0 = image_blocks + fimage_blocks;
    if ((int)blockIdx.x == check0 + 1 + a.rows) {
        __shared__ int red[2][256];
        // The rise of slot s: the largest sum of D~->D~ scores from it on (at
        // least 0, none), rise(s) = max(0, score into s + 1 + rise(s + 1)).  Each
        // thread takes neighbouring slots; what they make of the rise behind them
        // is max(own, sum + it), composed over the threads behind in log2(256)
        // steps.  A -inf score needs no case of its own: runs between them add
        // at most the range of D->M, less than it takes.  (A walk from every
        // slot instead, M = 2400 with D->D of 0: 12 ms a call.)
        constexpr int slots = 2 * G * Q, per = (slots + 255) / 256;
        const int s0 = (int)threadIdx.x * per;
        int sc[per], own = 0, sum = 0;
#pragma unroll
        for (int i = per - 1; i >= 0; --i) {
            const int s = s0 + i;             // score into slot s + 1
            sc[i] = s + 1 < slots ? (short)p7_slot_cost(a, a.rows + kFDD, s + 1) : kP7Neg;
            own = max(0, own + sc[i]);
            sum += sc[i];
        }
        __syncthreads();
        red[0][threadIdx.x] = own;
        red[1][threadIdx.x] = sum;
        __syncthreads();
        for (int h = 1; h < 256; h *= 2) {
            const int at = (int)threadIdx.x + h;
            const int o = at < 256 ? red[0][at] : 0, u = at < 256 ? red[1][at] : 0;
            __syncthreads();
            if (at < 256) {
                own = max(own, sum + o);
                sum += u;
                red[0][threadIdx.x] = own;
                red[1][threadIdx.x] = sum;
            }
            __syncthreads();
        }
        int r = (int)threadIdx.x < 255 ? red[0][threadIdx.x + 1] : 0;
#pragma unroll
        for (int i = per - 1; i >= 0; --i) {
            r = max(0, sc[i] + r);
            if (s0 + i < slots) a.rise[s0 + i] = r;
        }
        return;
    }
    if ((int)blockIdx.x > check0) {
        const int x = (int)blockIdx.x - check0 - 1;       // emission row
        bool big = false;
        if (x != kInvalidCode)
            for (int k = threadIdx.x; k < a.M; k += 256) big = big || a.msc[x * a.M + k] > kP7Bias;
        if (!__syncthreads_or(big) && threadIdx.x == 0) a.aux[kAuxEmisOk + x] = 1;
        else if (threadIdx.x == 0) a.aux[kAuxEmisOk + x] = 0;
        return;
    }
    if ((int)blockIdx.x == check0) {
        // the transitions: max of D->M, smallest I->I cost, and whether all are
        // within the bounds; and how many records the cost form takes.  (What
        // the latter needs from memory is read first.)
        __shared__ int red[2][256];
        __shared__ int gentle[kP7Loops];
        const int n = p7_records(a);
        const int step0 = (n + 255) / 256, r0 = (int)threadIdx.x * step0;
        const int probe = a.sel && r0 < n ? a.sel[r0] : a.nseq;
        if (threadIdx.x < kP7Loops) gentle[threadIdx.x] = (int)a.gentle[threadIdx.x];
        auto top = [&](int t) {                   // red[t][0] = the maximum
            __syncthreads();
            for (int h = 128; h > 0; h >>= 1) {
                if ((int)threadIdx.x < h && red[t][threadIdx.x + h] > red[t][threadIdx.x])
                    red[t][threadIdx.x] = red[t][threadIdx.x + h];
                __syncthreads();
            }
            return red[t][0];
        };
        int m = kP7Neg, mii = 65535;
        bool bad = a.tbm > 0 || a.tbm < -kP7MaxTbm;
        for (int k = threadIdx.x; k < a.M; k += 256) {
            const int dm = a.trans[5 * a.M + k], dd = a.trans[6 * a.M + k];
            const int ii = -(int)a.trans[4 * a.M + k];
            m = dm > m ? dm : m;
            mii = ii < mii ? ii : mii;
            bad = bad || (dm < -kP7MaxDm && dd > kP7Dead);
#pragma unroll
            for (int t = 0; t < 7; ++t) bad = bad || a.trans[t * a.M + k] > 0;
        }
        red[0][threadIdx.x] = m;
        red[1][threadIdx.x] = -mii;
        bad = __syncthreads_or(bad);
        const int maxdm = top(0), minii = -top(1);
        if (threadIdx.x == 0) {
            a.aux[kAuxMaxDm] = maxdm;
            a.aux[kAuxTransOk] = bad ? 0 : 1;
            a.aux[kAuxMinII] = minii;
        }
        // The records that the cost form takes: those whose |loop| is at most the
        // smallest I->I cost, the first ones of the processing order; of a
        // selection (longest first, as hmsv_select writes it), those before
        // the first position past them, found with 256 probes at a time.  In
        // any other order some of the rest are before it: the cost form's
        // kernel sends those back one by one.
        const int past = gentle[min(max(minii, 0), kP7Loops - 1)];
        int lo = a.sel ? 0 : min(past, n), hi = a.sel ? n : lo;
        while (lo < hi) {
            const bool whole = hi - lo == n;
            const int step = whole ? step0 : (hi - lo + 255) / 256;
            const int r = lo + (int)threadIdx.x * step;
            const int k = __syncthreads_count(r < hi && (whole ? probe : a.sel[r]) < past);
            hi = min(hi, lo + k * step);
            if (k > 0) lo += (k - 1) * step + 1;
        }
        if (threadIdx.x == 0) {
            a.aux[kAuxFast] = lo;
            a.aux[kAuxPend] = n - lo;             // the rest, listed first
        }
        if (threadIdx.x < kP7Parts) {                       // the record queues
            a.queue[threadIdx.x * 32] = 0u;
            a.fqueue[threadIdx.x * 32] = 0u;
        }
        return;
    }
    const bool cost = (int)blockIdx.x >= image_blocks;
    const int idx = (int)((blockIdx.x - (cost ? image_blocks : 0)) * 256 + threadIdx.x);
    if (idx >= (a.rows + (cost ? (int)kFRows : 7)) * D.RS) return;
    const int x = idx / D.RS;
    int rem = idx - x * D.RS;
    int w, q0;
    if (rem < D.OFF2) {
        const int ch = rem / D.CW;
        rem -= ch * D.CW;
        w = 4;
        q0 = ch * 4;
    } else if (rem < D.OFF1) {
        rem -= D.OFF2;
        w = 2;
        q0 = D.NF * 4;
    } else {
        rem -= D.OFF1;
        w = 1;
        q0 = D.NF * 4 + ((D.R & 2) ? 2 : 0);
    }
    rem %= G * w;
    const int jj = rem / w;
    const int qq = q0 + (rem - jj * w);
    const int s0 = qq + Q * (2 * jj);
    uint32_t v = 0u;
    if (qq < Q) {
        const uint32_t lo = cost ? p7_slot_cost(a, x, s0) : (uint16_t)(short)p7_slot_score(a, x, s0);
        const uint32_t hi = cost ? p7_slot_cost(a, x, s0 + Q)
                                 : (uint16_t)(short)p7_slot_score(a, x, s0 + Q);
        v = lo | (hi << 16);
    }
    (cost ? a.fimage : a.image)[idx] = v;
}

template <int G, int Q, int THREADS>
__global__ void __launch_bounds__(THREADS) p7_kernel(P7Args a) {
    using Lay = Layout<G, Q, kP7Rows>;
    constexpr int RS = Lay::RS;
    // Records: all of the call's, or, where the cost form holds for the profile,
    // the ones its kernel listed.
    const bool rest = p7_profile_fast(a);
    const int32_t *sel = rest ? a.pend : a.sel;
    const int nseq = rest ? a.aux[kAuxPend] : p7_records(a);
    if (rest) {
        // the first blocks are enough (at least one per queue)
        const int per = (int)(blockDim.x / G);
        const int need = (nseq + per - 1) / per;
        if (nseq == 0 || (int)blockIdx.x >= (need > kP7Parts ? need : kP7Parts)) return;
    }
    extern __shared__ uint32_t lds[];
    {
        const uint4 *src = (const uint4 *)a.image;
        uint4 *dst = (uint4 *)lds;
        const int n16 = (a.rows + 7) * (RS / 4);
        for (int i = threadIdx.x; i < n16; i += blockDim.x) dst[i] = src[i];
    }
    __syncthreads();
    const int maxdm = a.aux[kAuxMaxDm];       // max over nodes of D->M (prep kernel)

    const int lane = threadIdx.x & 63;
    const int j = lane % G;
    const bool gstart = j == 0;
    const uint32_t *T[3] = {lds + Lay::lane_off(lane, 4),
                            lds + Lay::OFF2 + Lay::lane_off(lane, 2),
                            lds + Lay::OFF1 + Lay::lane_off(lane, 1)};
    // Dwords of table row r for this lane: chunk ch of 4 (registers
    // 4ch..4ch+3), the 2-dword tail (registers Q2, Q2+1), the 1-dword tail
    // (register Q1).
    auto chunk = [&](uint32_t r, int ch) -> uint4 {
        return *(const uint4 *)((const char *)T[0] + r * (uint32_t)(RS * 4) + ch * Lay::CW * 4);
    };
    auto tail2 = [&](uint32_t r) -> uint2 {
        return *(const uint2 *)((const char *)T[1] + r * (uint32_t)(RS * 4));
    };
    auto tail1 = [&](uint32_t r) -> uint32_t {
        return *(const uint32_t *)((const char *)T[2] + r * (uint32_t)(RS * 4));
    };
    auto comp = [](const uint4 &v, int u) -> uint32_t {
        return u == 0 ? v.x : u == 1 ? v.y : u == 2 ? v.z : v.w;
    };
    const uint32_t rT = (uint32_t)a.rows;    // first transition row

    P7Queue<G> queue(a.queue, lane, j);
    auto take = [&]() -> int { return queue.take(sel, nseq); };

    s16x2 Mr[Q], Ir[Q], Dr[Q];
    queue.issue(true);
    int t = take();
    uint4 rec = make_uint4(0u, 0u, 0u, 0u), rec16 = rec;
    uint32_t lm = 0u;
    if (t >= 0) {
        rec = *(const uint4 *)(a.seqs + t);
        rec16 = *((const uint4 *)(a.seqs + t) + 1);
        lm = a.lenmodel[t];
    }
    // the next record, claimed and loaded while the current one runs
    queue.issue(true);
    int tn = take();
    uint4 nrec = rec, nrec16 = rec16;
    uint32_t nlm = lm;
    auto prefetch = [&]() {
        if (tn >= 0) {
            nrec = *(const uint4 *)(a.seqs + tn);
            nrec16 = *((const uint4 *)(a.seqs + tn) + 1);
            nlm = a.lenmodel[tn];
        }
    };

    bool active = false;
    uint32_t off = a.pad_off, seq_off = a.pad_off, id = 0;
    int len = 0, done = 0;       // residues of the sequence, rows run so far
    int loop = 0, move = 0;      // length model: N/J/C loops, N/J->B and C->T
    // special states, packed: JC = (J, C), NN = (N, N), B in Bv's low half
    s16x2 JC = splat16(kP7Neg), NN = splat16(0), Bv = splat16(0);
    s16x2 loop2 = splat16(0), move2 = splat16(0);
    const s16x2 tbm2 = splat16(a.tbm), half2 = splat16(kP7Half);
    bool ovf = false;
    uint4 wv = make_uint4(0u, 0u, 0u, 0u);   // this step's 16 residues
    const s16x2 neg = splat16(kP7Neg);
    auto start = [&]() {
        active = t >= 0;
        seq_off = active ? rec.x : a.pad_off;
        off = seq_off;
        id = rec.z;
        len = active ? (int)rec.w : 0;
        done = 0;
        loop = (int)(short)(lm & 0xffffu);
        move = (int)(short)(lm >> 16);
        loop2 = splat16(loop);
        move2 = splat16(move);
        NN = splat16(0);
        Bv = adds(NN, move2);
        JC = splat16(kP7Neg);
        ovf = false;
        wv = active ? rec16 : make_uint4(0x14141414u, 0x14141414u, 0x14141414u, 0x14141414u);
#pragma unroll
        for (int q = 0; q < Q; ++q) Mr[q] = Ir[q] = Dr[q] = neg;
    };
    start();
    prefetch();
    queue.issue(true);           // the record after that, taken at the switch

    for (;;) {
        if (!__any(active)) break;
        bool ended = false;
        do {
            // residues of the next step (the database stores every sequence
            // in whole 16-residue steps plus 16 more bytes)
            const uint4 wn = *(const uint4 *)(a.res + off + 16u);
            // The floor under the B->M score of the rows after this step's
            // rows (B >= N + move, and N only falls: the loop score is <= 0,
            // so N after the step's last row bounds every row of the step).
            // A D value d can raise a cell of the next row only through
            // D->M, to at most d + maxdm, while every such cell is at least
            // that floor: D values below thr cannot change any M, hence no E
            // and no score (D feeds nothing else).  A lower bound than the
            // row's own is still a bound, so one per step serves its rows.
            int thr_step;
            {
                const int nEnd = sat16((int)NN.x + 16 * loop);
                const int t1 = sat16(sat16(nEnd + move) + a.tbm) - maxdm - 1;
                thr_step = active ? (t1 > kP7Pos ? kP7Pos : (t1 < kP7Neg ? kP7Neg : t1)) : kP7Pos;
            }
            const s16x2 thr1 = splat16(thr_step);
#pragma unroll 1
            for (int r = 0; r < 16; ++r) {
                const uint32_t word = r < 4 ? wv.x : r < 8 ? wv.y : r < 12 ? wv.z : wv.w;
                const uint32_t x = __builtin_amdgcn_ubfe(word, 8u * (uint32_t)(r & 3), 8u);
                const bool live = active && done + r < len;
                const s16x2 bc = adds(__builtin_shufflevector(Bv, Bv, 0, 0), tbm2);
                // ---- M and I, registers in descending order ----------------
                // (in place: slot q's new M reads the old M, I and D of slot
                // q - 1, not yet overwritten; its new I reads its own old M
                // and I, updated first).  Slot 0 of each element reads the
                // previous element's last slot, shifted in before the pass.
                const s16x2 sM = as_s16x2(shift_in(s16_bits(Mr[Q - 1])));
                const s16x2 sI = as_s16x2(shift_in(s16_bits(Ir[Q - 1])));
                const s16x2 sD = as_s16x2(shift_in(s16_bits(Dr[Q - 1])));
                s16x2 xe = neg;
                auto mi_cell = [&](int q, uint32_t e, uint32_t mm, uint32_t im, uint32_t dm,
                                   uint32_t mi, uint32_t ii) {
                    const s16x2 gM = q > 0 ? Mr[q - 1] : sM;
                    const s16x2 gI = q > 0 ? Ir[q - 1] : sI;
                    const s16x2 gD = q > 0 ? Dr[q - 1] : sD;
                    // (pinned here: left to itself the compiler sinks the I
                    // update to the row's end and keeps copies of the old M)
                    s16x2 nI = smax(adds(Mr[q], as_s16x2(mi)), adds(Ir[q], as_s16x2(ii)));
                    asm volatile("" : "+v"(nI));
                    Ir[q] = nI;
                    const s16x2 c = smax(smax(adds(gM, as_s16x2(mm)), adds(gI, as_s16x2(im))),
                                         smax(adds(gD, as_s16x2(dm)), bc));
                    Mr[q] = adds(c, as_s16x2(e));
                    xe = smax(xe, Mr[q]);
                };
                if constexpr (Lay::T1) {
                    mi_cell(Lay::Q1, tail1(x), tail1(rT + kP7MMp), tail1(rT + kP7IMp),
                            tail1(rT + kP7DMp), tail1(rT + kP7MI), tail1(rT + kP7II));
                }
                if constexpr (Lay::T2) {
                    const uint2 ve = tail2(x), vmm = tail2(rT + kP7MMp), vim = tail2(rT + kP7IMp),
                                vdm = tail2(rT + kP7DMp), vmi = tail2(rT + kP7MI),
                                vii = tail2(rT + kP7II);
                    mi_cell(Lay::Q2 + 1, ve.y, vmm.y, vim.y, vdm.y, vmi.y, vii.y);
                    mi_cell(Lay::Q2, ve.x, vmm.x, vim.x, vdm.x, vmi.x, vii.x);
                }
#pragma unroll
                for (int ch = Lay::NF - 1; ch >= 0; --ch) {
                    // one chunk's 24 score dwords at a time: keeps the
                    // scheduler from hoisting every chunk's loads at once
                    __builtin_amdgcn_sched_barrier(0);
                    const uint4 ve = chunk(x, ch), vmm = chunk(rT + kP7MMp, ch),
                                vim = chunk(rT + kP7IMp, ch), vdm = chunk(rT + kP7DMp, ch),
                                vmi = chunk(rT + kP7MI, ch), vii = chunk(rT + kP7II, ch);
#pragma unroll
                    for (int u = 3; u >= 0; --u) {
                        if (ch * 4 + u < Q)
                            mi_cell(ch * 4 + u, comp(ve, u), comp(vmm, u), comp(vim, u),
                                    comp(vdm, u), comp(vmi, u), comp(vii, u));
                    }
                }
                // ---- D within each element, ascending ----------------------
                // (from the new M; slot 0 takes the previous element's last M
                // through M->D here, its last D below)
                const s16x2 sMn = as_s16x2(shift_in(s16_bits(Mr[Q - 1])));
                uint32_t dd0 = 0u;
                auto d_cell = [&](int q, uint32_t md, uint32_t dd) {
                    if (q == 0) {
                        Dr[0] = adds(sMn, as_s16x2(md));
                        dd0 = dd;
                    } else {
                        Dr[q] = smax(adds(Mr[q - 1], as_s16x2(md)), adds(Dr[q - 1], as_s16x2(dd)));
                    }
                };
#pragma unroll
                for (int ch = 0; ch < Lay::NF; ++ch) {
                    const uint4 vmd = chunk(rT + kP7MDp, ch), vdd = chunk(rT + kP7DDp, ch);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (ch * 4 + u < Q) d_cell(ch * 4 + u, comp(vmd, u), comp(vdd, u));
                }
                if constexpr (Lay::T2) {
                    const uint2 vmd = tail2(rT + kP7MDp), vdd = tail2(rT + kP7DDp);
                    d_cell(Lay::Q2, vmd.x, vdd.x);
                    d_cell(Lay::Q2 + 1, vmd.y, vdd.y);
                }
                if constexpr (Lay::T1) d_cell(Lay::Q1, tail1(rT + kP7MDp), tail1(rT + kP7DDp));
                // ---- D chains across elements, where they matter ----------
                // Each element's first slot takes the previous element's last
                // D (through D->D), carried along its slots; passes repeat
                // while some element's last D rose to a value that matters
                // (at least thr).  Values that do not matter may stay below
                // the sequential chain's.
                s16x2 in0 = adds(as_s16x2(shift_in(s16_bits(Dr[Q - 1]))), as_s16x2(dd0));
                s16x2 lim = smax(Dr[0], thr1);
                bool more = __any(s16_bits(smax(in0, lim)) != s16_bits(lim));
                while (more) {
                    const s16x2 last = Dr[Q - 1];
                    Dr[0] = smax(Dr[0], in0);
                    auto link = [&](int q, uint32_t dd) {
                        if (q > 0) Dr[q] = smax(Dr[q], adds(Dr[q - 1], as_s16x2(dd)));
                    };
#pragma unroll
                    for (int ch = 0; ch < Lay::NF; ++ch) {
                        const uint4 vdd = chunk(rT + kP7DDp, ch);
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (ch * 4 + u < Q) link(ch * 4 + u, comp(vdd, u));
                    }
                    if constexpr (Lay::T2) {
                        const uint2 vdd = tail2(rT + kP7DDp);
                        link(Lay::Q2, vdd.x);
                        link(Lay::Q2 + 1, vdd.y);
                    }
                    if constexpr (Lay::T1) link(Lay::Q1, tail1(rT + kP7DDp));
                    lim = smax(last, thr1);
                    more = __any(s16_bits(smax(Dr[Q - 1], lim)) != s16_bits(lim));
                    in0 = adds(as_s16x2(shift_in(s16_bits(Dr[Q - 1]))), as_s16x2(dd0));
                }
                // ---- special states (Plan-7 N, B, E, C, J) ----------------
                const int eh = (int)xe.x > (int)xe.y ? (int)xe.x : (int)xe.y;
                const int E = group_max<G>(eh);
                if (live) {
                    if (E >= kP7Pos) ovf = true;
                    // J = max(J + loop, E - 32), C = max(C + loop, E - 32)
                    JC = smax(adds(JC, loop2), adds(splat16(E), half2));
                    NN = adds(NN, loop2);
                    // B = max(N + move, J + move) = max(N, J) + move
                    // (saturation is monotone): the low halves
                    Bv = adds(smax(NN, JC), move2);
                }
            }
            done += 16;
            // groups without a sequence stay on the padding (>= 64 bytes of
            // code 20 at pad_off)
            if (active) off += 16u;
            wv = wn;
            ended = active && done >= len;
        } while (!__any(ended));

        // ---- finished sequences: score, then the next record ---------------
        if (ended && gstart) {
            a.score[id] = ovf ? (int16_t)kP7Pos : (int16_t)sat16((int)JC.y + move);
            a.flag[id] = ovf ? 1 : 0;
        }
        const int claimed = take();
        if (ended) {
            t = tn;
            tn = claimed;
            rec = nrec;
            rec16 = nrec16;
            lm = nlm;
            start();
            prefetch();
        }
        queue.issue(ended);
    }
}

}  // namespace hmsv
