// The Ising-machine stage of Alg. 3 on dense tiles, speculated: a span of
// positions is decided at once and repaired until it agrees with the
// sequential sweep (gfx950).
//
// A sweep visits the positions in order; position i is accepted iff
// dE_i + sum over the accepted k < i of 2 sigma_k sigma_i T[k][i] <= thr_i.
// Given any guess of the decisions of a span, evaluating every position of it
// against that guess and taking the answers as the next guess reaches a
// fixed point; the fixed point is the sequential sweep's, as position i's
// answer depends on lower positions only (by induction over i it is right
// after at most i + 1 rounds and stays).  Accepts are rare and a coupling is
// small beside the spread of dE, so almost every first guess is right: over
// spans of 64, 256 and 512 positions of post-Tabu sub-QUBOs the rounds that
// change anything are 1.4, 3.2 and 5.4 (m = 512, n = 5000), against 8, 31 and
// 62 accepts that a sweep taking accepts one at a time chains.
//
// Layout: one workgroup per (job, replica), one wave per block of 64
// positions (lane L of wave w owns position 64 w + L); a span is one block.
// The waves pass through MS phases per sweep, a barrier apart.  In phase b
// wave b settles its block and publishes its decisions in LDS, as 64 signed
// elements 2 sigma_k (k accepted) or 0; in the next phase every wave adds
// their products with its own lanes' columns of T, which stay in registers
// for the whole anneal: one dot instruction per four rows (two with int16
// couplings), whatever the number of accepts, the vector broadcast along
// each row of lanes by DPP from one LDS read per lane.  Meanwhile the next
// waves guess their decisions without the blocks still to come, so that
// when these arrive a wave mostly only confirms its own.
//
// Where a whole tile's columns do not fit the registers (mp = 1024, and mp =
// 512 with int16 couplings) a phase settles the NB blocks of one wave, which
// keeps the columns of its own and of the phase before's blocks only.  Other
// contributions go by accepted row: four more waves share out the accepted
// rows of a phase, read them whole from memory (16 bytes a lane, all MS
// blocks' columns), sum them in registers, and add their sums for a phase's
// blocks to these blocks' fields in LDS while the phase before it runs.
//
// What bounds it is latency: from one phase to the next an LDS exchange over
// a barrier (200 cycles), 16 dots (110), a comparison and, where a guess was
// wrong, a round more (about 250).  One sweep, 256 jobs, R = 1, int8, against
// the kernels that chain the accepts one by one: m = 64 0.55 us (1.5),
// 128 0.8 us (1.9), 256 1.5 us (3.4), 512 2.9 us (6.7), 1024 8 us (23).
// Measured and left out: deciding two or four blocks as one span over a
// barrier per round (m = 512: 4.5 ms per 1000 sweeps against 3.0), and
// correcting a published guess by single rows in place of the 16 dots (3.9).
#include <algorithm>

#include "qb_internal.h"

namespace {

template <typename TT, int MS>
struct Spec {
    static constexpr bool I8 = sizeof(TT) == 1;
    static constexpr int DW = I8 ? 16 : 32;                    // dwords of 64 couplings
    static constexpr bool ALL = MS <= (I8 ? 8 : 4);            // the whole tile's columns in registers
    static constexpr int NB = !ALL && I8 ? 2 : 1;              // blocks per wave and phase
    static constexpr int NP = MS / NB;                         // phases, and waves with blocks
    static constexpr int FW = ALL ? 0 : 4;                     // waves that read rows
    static constexpr int NT = 64 * (NP + FW);
    static constexpr int RW = MS * (int)sizeof(TT) / 4;        // dwords of a row per lane
    static constexpr int P = NP < 4 / NB ? NP : 4 / NB;        // sweeps per Philox call of a wave
    // one block's column: a vector, so that an index into it stays in registers
    using Col = uint32_t __attribute__((ext_vector_type(DW)));
};

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel)
{
    return (uint32_t)__builtin_amdgcn_perm(hi, lo, sel);
}

// 16 dots of the wave's column dwords t with the vector whose dword i is in
// lane i of every row of 16 lanes, in two chains.  One ALU sequence: the
// compiler would broadcast by a separate move per dword.  (Two wait states
// before a DPP read of a fresh register, three after a dot before another
// kind of instruction touches its result.)
#define QB_DOT(OP, D, T, L) OP " " D ", %2, " T " row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t"
#define QB_SPEC_DOTS(OP)                                                                                               \
    asm("s_nop 1\n\t" QB_DOT(OP, "%0", "%3", "0") QB_DOT(OP, "%1", "%4", "1") QB_DOT(OP, "%0", "%5", "2")              \
            QB_DOT(OP, "%1", "%6", "3") QB_DOT(OP, "%0", "%7", "4") QB_DOT(OP, "%1", "%8", "5")                         \
                QB_DOT(OP, "%0", "%9", "6") QB_DOT(OP, "%1", "%10", "7") QB_DOT(OP, "%0", "%11", "8")                   \
                    QB_DOT(OP, "%1", "%12", "9") QB_DOT(OP, "%0", "%13", "10") QB_DOT(OP, "%1", "%14", "11")            \
                        QB_DOT(OP, "%0", "%15", "12") QB_DOT(OP, "%1", "%16", "13") QB_DOT(OP, "%0", "%17", "14")       \
                            QB_DOT(OP, "%1", "%18", "15") "s_nop 2"                                                     \
        : "+v"(acc), "+v"(acc2)                                                                                        \
        : "v"(vec), "v"(t[O]), "v"(t[O + 1]), "v"(t[O + 2]), "v"(t[O + 3]), "v"(t[O + 4]), "v"(t[O + 5]),              \
          "v"(t[O + 6]), "v"(t[O + 7]), "v"(t[O + 8]), "v"(t[O + 9]), "v"(t[O + 10]), "v"(t[O + 11]),                  \
          "v"(t[O + 12]), "v"(t[O + 13]), "v"(t[O + 14]), "v"(t[O + 15]))

template <bool I8, int O, typename Col>
__device__ __forceinline__ int32_t dots16(int32_t acc, uint32_t vec, const Col &t)
{
    int32_t acc2 = 0;
    if constexpr (I8)
        QB_SPEC_DOTS("v_dot4c_i32_i8_dpp");
    else
        QB_SPEC_DOTS("v_dot2c_i32_i16_dpp");
    return acc + acc2;
}
#undef QB_SPEC_DOTS
#undef QB_DOT

// The lane's dwords of a 64-bit mask as element masks: with int8 couplings
// dword lane & 15 covers positions 4 (lane & 15) ..., one byte each; with
// int16 ones dwords lane & 15 and 16 + (lane & 15) two positions each.
template <bool I8>
struct MaskVec {
    uint32_t v[I8 ? 1 : 2];
};
template <bool I8>
__device__ __forceinline__ MaskVec<I8> expand(uint64_t mask, int lane)
{
    MaskVec<I8> r;
    const int l = lane & 15;
    if constexpr (I8) {
        const uint32_t half = l & 8 ? (uint32_t)(mask >> 32) : (uint32_t)mask;
        const uint32_t nib = (half >> (4 * (l & 7))) & 15u;
        // bit j of the nibble to byte j, and 1 to 0xFF (byte selectors 0x0C
        // and 0x0D of v_perm are 0x00 and 0xFF)
        r.v[0] = perm(0u, 0u, (__umul24(nib, 0x00204081u) & 0x01010101u) | 0x0C0C0C0Cu);
    } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t two = (h ? (uint32_t)(mask >> 32) : (uint32_t)mask) >> (2 * l);
            const uint32_t t = (two & 1u) | ((two & 2u) << 15);
            r.v[h] = perm(0u, 0u, (t << 8 | t) | 0x0C0C0C0Cu);
        }
    }
    return r;
}

// acc + column . vector of one block
template <bool I8, typename Col>
__device__ __forceinline__ int32_t block_dot(int32_t acc, const MaskVec<I8> &v, const Col &t)
{
    acc = dots16<I8, 0>(acc, v.v[0], t);
    if constexpr (!I8) acc = dots16<I8, 16>(acc, v.v[1], t);
    return acc;
}

// 2 sigma per element from the mask of spins set
template <bool I8>
__device__ __forceinline__ MaskVec<I8> signs(uint64_t ymask, int lane)
{
    MaskVec<I8> y = expand<I8>(ymask, lane);
#pragma unroll
    for (int h = 0; h < (I8 ? 1 : 2); ++h) y.v[h] = I8 ? 0x02020202u ^ (y.v[h] & 0xFCFCFCFCu) : 0x00020002u ^ (y.v[h] & 0xFFFCFFFCu);
    return y;
}

// Couplings of the lane's position with the blocks b0 .. b0 + NB - 1, packed
// along the rows of each block: t[v][i] holds rows 64 (b0 + v) + PER i ...
// The tile is symmetric, so the lane's column is its own row `row`, whose
// element (L, s) lies at L MS + s.
template <typename TT, int MS, int NB>
__device__ __forceinline__ void load_columns(const TT *__restrict__ row, int b0,
                                             typename Spec<TT, MS>::Col (&t)[NB])
{
    constexpr int DW = Spec<TT, MS>::DW;
    if constexpr (sizeof(TT) == 1) {
        const uint8_t *p = reinterpret_cast<const uint8_t *>(row);
#pragma unroll
        for (int i = 0; i < DW; ++i) {
            if constexpr (MS == 1) {
                t[0][i] = *reinterpret_cast<const uint32_t *>(p + 4 * i);
            } else if constexpr (MS == 2) {
                const uint2 d = *reinterpret_cast<const uint2 *>(p + 8 * i);
                t[0][i] = perm(d.y, d.x, 0x06040200u);
                t[1][i] = perm(d.y, d.x, 0x07050301u);
            } else {
                static_assert(NB % 4 == 0, "whole quads");
#pragma unroll
                for (int qd = 0; qd < NB / 4; ++qd) {
                    uint32_t w[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        w[r] = *reinterpret_cast<const uint32_t *>(p + (4 * i + r) * MS + b0 + 4 * qd);
                    const uint32_t l01 = perm(w[1], w[0], 0x05010400u), h01 = perm(w[1], w[0], 0x07030602u);
                    const uint32_t l23 = perm(w[3], w[2], 0x05010400u), h23 = perm(w[3], w[2], 0x07030602u);
                    t[4 * qd + 0][i] = perm(l23, l01, 0x05040100u);
                    t[4 * qd + 1][i] = perm(l23, l01, 0x07060302u);
                    t[4 * qd + 2][i] = perm(h23, h01, 0x05040100u);
                    t[4 * qd + 3][i] = perm(h23, h01, 0x07060302u);
                }
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < DW; ++i) {
            if constexpr (MS == 1) {
                t[0][i] = *reinterpret_cast<const uint32_t *>(row + 2 * i);
            } else {
#pragma unroll
                for (int pr = 0; pr < NB / 2; ++pr) {
                    const uint32_t w0 = *reinterpret_cast<const uint32_t *>(row + (2 * i) * MS + b0 + 2 * pr);
                    const uint32_t w1 = *reinterpret_cast<const uint32_t *>(row + (2 * i + 1) * MS + b0 + 2 * pr);
                    t[2 * pr + 0][i] = perm(w1, w0, 0x05040100u);
                    t[2 * pr + 1][i] = perm(w1, w0, 0x07060302u);
                }
            }
        }
    }
}

// The same for the NB blocks from b0 on, at mp >= 512: an element or a pair
// of elements at a time.
template <typename TT, int MS>
__device__ __forceinline__ void load_columns_of(const TT *__restrict__ row, int b0,
                                                typename Spec<TT, MS>::Col (&t)[Spec<TT, MS>::NB])
{
    using Pair = uint16_t;
    static_assert(Spec<TT, MS>::NB * sizeof(TT) == sizeof(Pair), "NB elements are two bytes");
#pragma unroll
    for (int i = 0; i < Spec<TT, MS>::DW; ++i) {
        if constexpr (sizeof(TT) == 1) {
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = *reinterpret_cast<const Pair *>(row + (4 * i + j) * MS + b0);
            const uint32_t l = w[0] | (w[1] << 16), h = w[2] | (w[3] << 16);
            t[0][i] = perm(h, l, 0x06040200u);
            t[1][i] = perm(h, l, 0x07050301u);
        } else {
            t[0][i] = (uint32_t)*reinterpret_cast<const Pair *>(row + 2 * i * MS + b0) |
                      ((uint32_t)*reinterpret_cast<const Pair *>(row + (2 * i + 1) * MS + b0) << 16);
        }
        // (a few loads at a time: a wave has 168 registers, and MS = 16 of int8
        // spills 141 words a lane as it is, MS = 8 of int16 20)
        if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
}

// A column's rows below the lane.
template <typename TT, int MS>
__device__ __forceinline__ typename Spec<TT, MS>::Col below(const typename Spec<TT, MS>::Col &t, int lane)
{
    constexpr int PER = 4 / (int)sizeof(TT), EB = 32 / PER;
    typename Spec<TT, MS>::Col r;
#pragma unroll
    for (int i = 0; i < Spec<TT, MS>::DW; ++i) {
        const int n = min(max(lane - PER * i, 0), PER);
        r[i] = n == PER ? t[i] : t[i] & ((1u << (EB * n)) - 1u);
    }
    return r;
}

// Bits of a mask below the lane.
__device__ __forceinline__ int below_count(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// A wave's blocks and its replica's random numbers.
template <int MS, typename TT>
struct SpecWave {
    using C = Spec<TT, MS>;
    static constexpr int NB = C::NB, P = C::P, PW = P * NB;   // blocks of a Philox call
    static constexpr bool I8 = C::I8;
    using Thr = int32_t[2][P][MS][64];   // thresholds of P sweeps, double-buffered

    int lane, w, nsw, B, r;
    const int32_t *thr;
    uint32_t k0, k1, tag;
    bool real[NB];                       // the lane's positions lie in the job
    int32_t F[NB], M[NB];                // flip basis; -y
    int64_t e = 0;
    int32_t nacc = 0;
    typename C::Col TL[NB];              // the own blocks' columns below the lane
    // while the blocks are open: thresholds, what their own decisions so far
    // make of the field, these, and 2 sigma of the elements that the lane expands
    int32_t tk[NB], own[NB];
    uint64_t acc[NB];
    MaskVec<I8> sg[NB];

    // thresholds of sweep sw0 + (w mod P) for the blocks of the wave's Philox
    // group: every wave makes one call per P sweeps and uses all of it
    __device__ __forceinline__ void thresholds(int sw0, int32_t (&tv)[PW])
    {
        const int sw = sw0 + w % P;
        if (sw < nsw) {
            const uint4 o = qb_philox(make_uint4(((uint32_t)(w * NB / 4) << 6) | (uint32_t)lane, (uint32_t)sw,
                                                 (uint32_t)r, tag), k0, k1);
#pragma unroll
            for (int i = 0; i < PW; ++i) tv[i] = thr[((size_t)sw << B) + (qb_word(o, i) >> (32 - B))];
        }
    }
    __device__ __forceinline__ void put(Thr &tb, int buf, const int32_t (&tv)[PW])
    {
#pragma unroll
        for (int i = 0; i < PW; ++i) tb[buf][w % P][(w / P) * PW + i][lane] = tv[i];
    }
    __device__ __forceinline__ void open(const Thr &tb, int sw)
    {
        // a lane past the job never accepts: no dE reaches INT32_MIN (|dE| <=
        // |F| < 2^31, checked when the problem is created)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            tk[j] = tb[(sw / P) & 1][sw % P][w * NB + j][lane];
            if (!real[j]) tk[j] = INT32_MIN;
            own[j] = 0;
            acc[j] = 0;
            sg[j] = signs<I8>(__ballot(M[j] != 0), lane);
        }
    }
    __device__ __forceinline__ int32_t dE(int j) const { return ((F[j] + own[j]) ^ M[j]) - M[j]; }
    __device__ __forceinline__ MaskVec<I8> own_vec(int j) const
    {
        MaskVec<I8> a = expand<I8>(acc[j], lane);
#pragma unroll
        for (int h = 0; h < (I8 ? 1 : 2); ++h) a.v[h] &= sg[j].v[h];
        return a;
    }
    // one round of block j, whose field has `add` besides; false once it is
    // at its fixed point
    __device__ __forceinline__ bool refine(int j, int32_t add = 0)
    {
        const uint64_t n = __ballot(dE(j) <= tk[j]);
        if (n == acc[j]) return false;
        acc[j] = n;
        own[j] = block_dot<I8>(add, own_vec(j), TL[j]);
        return true;
    }
    __device__ __forceinline__ bool mine(int j) const { return __builtin_amdgcn_inverse_ballot_w64(acc[j]); }
    __device__ __forceinline__ void publish(int j, TT *vec) const { vec[lane] = (TT)(mine(j) ? (M[j] ? -2 : 2) : 0); }
    // energy, count and spins of a settled block
    __device__ __forceinline__ void close(int j)
    {
        e += mine(j) ? dE(j) : 0;
        nacc += __builtin_popcountll(acc[j]);
        M[j] ^= mine(j) ? -1 : 0;
    }
};

// Columns in registers: every published vector is added by every wave.  A
// job of m variables has ceil(m / 64) blocks, and as many phases.
template <int MS, typename TT>
__device__ __forceinline__ void spec_sweeps(SpecWave<MS, TT> &S, const TT *__restrict__ row, int nblocks,
                                            typename SpecWave<MS, TT>::Thr &tb)
{
    using C = Spec<TT, MS>;
    constexpr int DW = C::DW, P = C::P, HV = C::I8 ? 1 : 2;
    __shared__ __align__(16) TT vec[2][64];          // published decisions, by phase parity
    const int w = S.w, lane = S.lane, nsw = S.nsw;
    // the own block's column is split at the diagonal: the rows below the
    // lane enter its decision (TL), the others its field afterwards
    typename C::Col T[MS];
    load_columns<TT, MS, MS>(row, 0, T);
#pragma unroll
    for (int v = 0; v < MS; ++v)
        if (v == w) {
            S.TL[0] = below<TT, MS>(T[v], lane);
#pragma unroll
            for (int i = 0; i < DW; ++i) T[v][i] ^= S.TL[0][i];
        }
    int32_t tvn[P] = {};
    S.thresholds(0, tvn);
    S.put(tb, 0, tvn);
    __syncthreads();
    constexpr int AHEAD = MS == 2 ? 1 : MS == 4 ? 2 : 3;
    if (w <= AHEAD) S.open(tb, 0);
    int par = 0;                                     // of the sweep's first phase
#pragma unroll 1
    for (int sw = 0; sw < nsw; ++sw) {
        const bool fresh = sw % P == 0;
        if (fresh) S.thresholds(sw + P, tvn);
        if constexpr (MS == 1) {
            while (S.refine(0)) {}
            S.close(0);
            S.F[0] = block_dot<C::I8>(S.F[0] + S.own[0], S.own_vec(0), T[0]);
            S.put(tb, (sw & 1) ^ 1, tvn);
            S.open(tb, sw + 1);
        } else {
#pragma unroll
            for (int b = 0; b < MS; ++b) {
                // (opaque: the phases' comparisons are cheaper made anew than
                // kept for all phases, which spills)
                int w = S.w, nb = nblocks;
                asm volatile("" : "+s"(w), "+s"(nb));
                if (b > MS / 2 && b >= nb) break;
                if (b > 0 || sw > 0) {
                    qb_lds_barrier();
                    const int bp = b > 0 ? b - 1 : nb - 1;
                    MaskVec<C::I8> v;
#pragma unroll
                    for (int h = 0; h < HV; ++h) v.v[h] = reinterpret_cast<const uint32_t *>(vec[par ^ (b & 1) ^ 1])[16 * h + (lane & 15)];
                    if (w == bp) {
                        S.close(0);
                        S.F[0] += S.own[0];
                    }
#pragma unroll
                    for (int c = b > 0 ? b - 1 : MS / 2; c < (b > 0 ? b : MS); ++c)
                        if (b > 0 || c == nb - 1) S.F[0] = block_dot<C::I8>(S.F[0], v, T[c]);
                }
                if (w == b) {
                    while (S.refine(0)) {}
                    S.publish(0, vec[par ^ (b & 1)]);
                    __builtin_amdgcn_s_setprio(0);
                }
                // the next waves: one round each per phase, so that they are
                // never what the phase waits for
#pragma unroll
                for (int d = AHEAD; d >= 1; --d) {
                    const bool wrap = b + d >= nb;
                    if (w == b + d - (wrap ? nb : 0)) {
                        if (d == AHEAD) S.open(tb, wrap ? sw + 1 : sw);
                        if (d < AHEAD || MS == 2) S.refine(0);
                        // a phase is as long as its settling wave takes: that one first
                        if (MS > 4 && d == 1) __builtin_amdgcn_s_setprio(3);
                    }
                }
            }
            par ^= nblocks & 1;
            if (fresh) S.put(tb, ((sw / P) & 1) ^ 1, tvn);
        }
    }
    if (MS > 1 && w == nblocks - 1) S.close(0);
}

// A row-reading wave's sums, per block: the lane's elements of a row are the
// MS blocks' columns.  int8 couplings: biased by 128 (127 in a row taken
// negative, whose bits are inverted), two 16-bit sums a register, all modulo
// 2^16 and relative to the running total of the biases (a block's sum is
// taken once a sweep, over at most 257 rows: |sum| < 2^15).
template <typename TT, int MS>
struct RowSums {
    static constexpr bool I8 = sizeof(TT) == 1;
    static constexpr int RW = Spec<TT, MS>::RW, PER = 4 / (int)sizeof(TT), EB = 32 / PER;
    using U16x2 = uint16_t __attribute__((ext_vector_type(2)));
    uint32_t sum[I8 ? MS / 2 : MS] = {};
    uint32_t bias = 0;                               // uniform

    // adds a row, but for the blocks s0 .. s0 + NB - 1
    template <int NB>
    __device__ __forceinline__ void add(const uint4 &row, bool neg, int s0)
    {
        static_assert(RW == 4, "16 bytes a lane");
        const uint32_t r[4] = {row.x, row.y, row.z, row.w};
        const uint32_t flip = neg ? 0x7F7F7F7Fu : 0x80808080u;
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            uint32_t keep = ~0u;
#pragma unroll
            for (int n = 0; n < NB; ++n)
                if ((s0 + n) / PER == i) keep &= ~((0xFFFFFFFFu >> (32 - EB)) << (EB * ((s0 + n) % PER)));
            if constexpr (I8) {
                const uint32_t y = (r[i] & keep) ^ flip;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const U16x2 z = __builtin_bit_cast(U16x2, perm(0u, y, h ? 0x0C030C01u : 0x0C020C00u));
                    const U16x2 t = __builtin_bit_cast(U16x2, sum[2 * i + h]);
                    sum[2 * i + h] = __builtin_bit_cast(uint32_t, (U16x2)(t + z));
                }
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int32_t x = (int32_t)((r[i] & keep) << (h ? 0 : 16)) >> 16;
                    sum[2 * i + h] += (uint32_t)(neg ? -x : x);
                }
            }
        }
        if (I8) bias += neg ? 127u : 128u;
    }
    // block s's sum, which starts again
    __device__ __forceinline__ int32_t take(int s)
    {
        if constexpr (I8) {
            uint32_t &t = sum[2 * (s / 4) + (s & 1)];
            const int sh = s & 2 ? 16 : 0;
            const int32_t x = (int32_t)(int16_t)(uint16_t)((t >> sh) - bias);
            t = (t & (0xFFFF0000u >> sh)) | ((bias & 0xFFFFu) << sh);
            return x;
        } else {
            const int32_t x = (int32_t)sum[s];
            sum[s] = 0;
            return x;
        }
    }
};

// What the waves of a replica share where rows are read from memory.
template <typename TT, int MS>
struct FarLds {
    static constexpr int NB = Spec<TT, MS>::NB;
    // by phase parity: decisions as elements; accepted rows with their sign, and their number
    TT vec[2][NB][64];
    uint32_t list[2][128];
    int32_t cnt[2];
    int32_t far[MS][64];                             // fields' part from rows
};

template <int MS, typename TT>
__device__ __forceinline__ void spec_rows(int f, int lane, int nsw, int np, const TT *__restrict__ tile, FarLds<TT, MS> &L)
{
    using C = Spec<TT, MS>;
    constexpr int NB = C::NB, NP = C::NP, FW = C::FW, MP = 64 * MS, U = 8;
    RowSums<TT, MS> sums;
    const TT *col = tile + lane * MS;
    int par = 0;
#pragma unroll 1
    for (int sw = 0; sw < nsw; ++sw) {
#pragma unroll
        for (int b = 0; b < NP; ++b) {
            if (b >= np) break;
            if (b > 0 || sw > 0) {
                qb_lds_barrier();
                const uint32_t lo = L.list[par ^ 1][lane], hi = NB > 1 ? L.list[par ^ 1][64 + lane] : 0u;
                const int cnt = __builtin_amdgcn_readfirstlane(L.cnt[par ^ 1]);
                for (int i0 = f; i0 < cnt; i0 += U * FW) {
                    uint4 x[U];
                    uint32_t en[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = i0 + u * FW;
                        if (i < cnt) {
                            en[u] = (uint32_t)(i < 64 ? __builtin_amdgcn_readlane((int)lo, i)
                                                      : __builtin_amdgcn_readlane((int)hi, i - 64));
                            x[u] = *reinterpret_cast<const uint4 *>(col + (size_t)(en[u] & 0xFFFFu) * MP);
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (i0 + u * FW < cnt) sums.template add<NB>(x[u], en[u] >> 16 != 0, b * NB);
                }
            }
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                const bool wrap = b + 1 == np;
                const int32_t x = wrap ? sums.take(n) : sums.take(((b + 1) % NP) * NB + n);
                if (__ballot(x != 0)) atomicAdd(&L.far[wrap ? n : (b + 1) * NB + n][lane], 2 * x);
            }
            par ^= 1;
        }
    }
}

// Near blocks' columns in registers, farther rows by spec_rows.
template <int MS, typename TT>
__device__ __forceinline__ void spec_sweeps_far(SpecWave<MS, TT> &S, const TT *__restrict__ tile, int np,
                                                typename SpecWave<MS, TT>::Thr &tb, FarLds<TT, MS> &L)
{
    using C = Spec<TT, MS>;
    constexpr int NB = C::NB, NP = C::NP, P = C::P, HV = C::I8 ? 1 : 2, MP = 64 * MS;
    const int w = S.w, lane = S.lane, nsw = S.nsw;
    // columns of the NB blocks before with the wave's blocks, and of its first with its second
    typename C::Col N[NB][NB], X;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const TT *row = tile + (size_t)(64 * (w * NB + j) + lane) * MP;
        typename C::Col t[NB];
        load_columns_of<TT, MS>(row, w * NB, t);
        S.TL[j] = below<TT, MS>(t[j], lane);
        if (j == 1) X = t[0];
        load_columns_of<TT, MS>(row, (w > 0 ? w - 1 : np - 1) * NB, N[j]);
    }
    int32_t tvn[SpecWave<MS, TT>::PW] = {};
    S.thresholds(0, tvn);
    S.put(tb, 0, tvn);
    __syncthreads();
    if (w == 0) S.open(tb, 0);
    int due = -1;                                    // buffer that waits for the thresholds in tvn
    int par = 0;
#pragma unroll 1
    for (int sw = 0; sw < nsw; ++sw) {
#pragma unroll 1
        for (int b = 0; b < np; ++b) {
            // phases to go until the wave settles (np > 4); one past the job's
            // blocks only makes thresholds
            const int d = w >= np ? 3 - b : w - b + (w < b ? np : 0);
            const bool begun = b > 0 || sw > 0;
            // a phase is as long as its settling wave takes: that one first
            if (d == 0 && w < np) __builtin_amdgcn_s_setprio(3);
            if (begun) qb_lds_barrier();
            if (w >= np && d < 2) {
            } else if (d == 0) {
#pragma unroll
                for (int j = 0; j < NB; ++j) S.F[j] += L.far[w * NB + j][lane];
                if (begun) {
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        MaskVec<C::I8> v;
                        const uint32_t *p = reinterpret_cast<const uint32_t *>(L.vec[par ^ 1][i]);
#pragma unroll
                        for (int h = 0; h < HV; ++h) v.v[h] = p[16 * h + (lane & 15)];
#pragma unroll
                        for (int j = 0; j < NB; ++j) S.F[j] = block_dot<C::I8>(S.F[j], v, N[j][i]);
                    }
                }
                while (S.refine(0)) {}
                S.publish(0, L.vec[par][0]);
                int n = __builtin_popcountll(S.acc[0]);
                if constexpr (NB == 2) {
                    const int32_t cross = S.acc[0] ? block_dot<C::I8>(0, S.own_vec(0), X) : 0;
                    S.own[1] = cross;
                    while (S.refine(1, cross)) {}
                    S.publish(1, L.vec[par][1]);
                    if (S.mine(1)) L.list[par][n + below_count(S.acc[1])] = (uint32_t)(64 * (2 * w + 1) + lane) | (S.M[1] ? 0x10000u : 0u);
                    n += __builtin_popcountll(S.acc[1]);
                }
                if (S.mine(0)) L.list[par][below_count(S.acc[0])] = (uint32_t)(64 * NB * w + lane) | (S.M[0] ? 0x10000u : 0u);
                if (lane == 0) L.cnt[par] = n;
#pragma unroll
                for (int j = 0; j < NB; ++j) L.far[w * NB + j][lane] = 0;
                __builtin_amdgcn_s_setprio(0);
            } else if (d == 1) {
                S.open(tb, b + 1 < np ? sw : sw + 1);
            } else if (d == np - 1 && w < np) {
                if (begun) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) S.close(j);
                }
            } else if (d == 3) {
                if (sw % P == 0) {
                    S.thresholds(sw + P, tvn);
                    due = (sw / P + 1) & 1;
                }
            } else if (d == 2 && due >= 0) {
                S.put(tb, due, tvn);
                due = -1;
            }
            par ^= 1;
        }
    }
    if (w == np - 1) {
#pragma unroll
        for (int j = 0; j < NB; ++j) S.close(j);
    }
}

template <int MS, typename TT>
__device__ __forceinline__ void anneal_spec_item(int item, const int32_t *__restrict__ jobs,
                                                 const int32_t *__restrict__ off, const int64_t *__restrict__ tile_off,
                                                 const TT *__restrict__ tiles, const int32_t *__restrict__ F0,
                                                 const uint8_t *__restrict__ y0, int nsw, int B,
                                                 const int32_t *__restrict__ thr, int R, uint32_t k0, uint32_t k1,
                                                 uint32_t inst_base, const qb_iter *__restrict__ it,
                                                 uint8_t *__restrict__ Y, int64_t *__restrict__ eout,
                                                 int32_t *__restrict__ acnt)
{
    __shared__ typename SpecWave<MS, TT>::Thr tb;
    __shared__ int64_t esum[Spec<TT, MS>::NP];
    __shared__ int32_t asum[Spec<TT, MS>::NP];
    const int q = jobs[item / R], r = item % R;
    const int base = off[q], m = off[q + 1] - base;
    const TT *gt = tiles + tile_off[q];
    FarLds<TT, MS> *far = nullptr;
    using C = Spec<TT, MS>;
    constexpr int NB = C::NB, NP = C::NP;
    const int np = (m + 64 * NB - 1) / (64 * NB);    // phases that the job needs
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if constexpr (!C::ALL) {
        __shared__ __align__(16) FarLds<TT, MS> L;
        for (int t = threadIdx.x; t < MS * 64; t += C::NT) (&L.far[0][0])[t] = 0;
        if (w >= NP) {
            __syncthreads();
            spec_rows<MS, TT>(w - NP, lane, nsw, np, gt, L);
            __syncthreads();
            return;
        }
        far = &L;
    }
    SpecWave<MS, TT> S;
    S.lane = lane;
    S.w = w;
    S.nsw = nsw;
    S.B = B;
    S.r = r;
    S.thr = thr;
    S.k0 = k0;
    S.k1 = k1;
    S.tag = (1u << 28) | (inst_base + (it ? it->inst : 0u) + (uint32_t)q);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int pos = 64 * (w * NB + j) + lane;
        S.real[j] = pos < m;
        S.F[j] = S.real[j] ? F0[base + pos] : 0;
        S.M[j] = (S.real[j] && y0[base + pos]) ? -1 : 0;
    }
    if constexpr (C::ALL)
        spec_sweeps<MS, TT>(S, gt + (size_t)(64 * w + lane) * (64 * MS), (m + 63) / 64, tb);
    else
        spec_sweeps_far<MS, TT>(S, gt, np, tb, *far);
#pragma unroll
    for (int j = 0; j < NB; ++j)
        if (S.real[j]) Y[(size_t)base * R + (size_t)r * m + 64 * (w * NB + j) + lane] = (uint8_t)(S.M[j] & 1);
    const int64_t e = qb_wave_sum_i64(S.e);
    if (lane == 0) {
        esum[w] = e;
        asum[w] = S.nacc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        int32_t na = 0;
        for (int v = 0; v < NP; ++v) {
            t += esum[v];
            na += asum[v];
        }
        eout[(size_t)q * R + r] = t;
        if (acnt) acnt[(size_t)q * R + r] = na;
    }
}

template <int MS, typename TT>
__global__ void __launch_bounds__((Spec<TT, MS>::NT))
    k_anneal_spec(const int32_t *__restrict__ jobs, const int32_t *__restrict__ off,
                  const int64_t *__restrict__ tile_off, const TT *__restrict__ tiles, const int32_t *__restrict__ F0,
                  const uint8_t *__restrict__ y0, int nsw, int B, const int32_t *__restrict__ thr, int R, uint32_t k0,
                  uint32_t k1, uint32_t inst_base, const qb_iter *__restrict__ it, uint8_t *__restrict__ Y,
                  int64_t *__restrict__ eout, int32_t *__restrict__ acnt, int *__restrict__ queue, int nitems)
{
    __shared__ int slot_s;
    for (int pass = 0;; ++pass) {
        const int item = qb_next_slot(queue, nitems, pass, &slot_s);
        if (item < 0) break;
        anneal_spec_item<MS, TT>(item, jobs, off, tile_off, tiles, F0, y0, nsw, B, thr, R, k0, k1, inst_base, it, Y,
                                 eout, acnt);
        __syncthreads();   // the next item reuses the workgroup's LDS
    }
}

template <int MS, typename TT>
void launch(int grid, hipStream_t s, const int32_t *jobs, qb_batch b, const void *tiles, const int32_t *F0,
            const uint8_t *y0, int nsw, int B, const int32_t *thr, int R, uint64_t seed, uint32_t inst_base,
            const qb_iter *it, uint8_t *Y, int64_t *e, int nitems)
{
    k_anneal_spec<MS, TT><<<grid, Spec<TT, MS>::NT, 0, s>>>(jobs, b->off_d, b->tile_off_d, (const TT *)tiles, F0, y0, nsw, B,
                                                   thr, R, (uint32_t)seed, (uint32_t)(seed >> 32), inst_base, it, Y, e,
                                                   b->acnt_d, b->lq, nitems);
}

}  // namespace

// One size class: a workgroup per (job, replica), or the persistent grid
// pulling them from the class's queue.  False for the one class without a
// kernel here: mp = 1024 with int16 couplings, whose columns do not fit.
bool qb_launch_anneal_spec(int cls, bool int8_tile, int njobs, int R, hipStream_t s, const int32_t *jobs, qb_batch b,
                           const void *tiles, const int32_t *F0, const uint8_t *y0, int nsw, int B, const int32_t *thr,
                           uint64_t seed, uint32_t inst_base, const qb_iter *it, uint8_t *Y, int64_t *e)
{
    const int nitems = njobs * R;
    const int grid = b->lgrid ? std::min(b->lgrid, nitems) : nitems;
#define QB_ARGS grid, s, jobs, b, tiles, F0, y0, nsw, B, thr, R, seed, inst_base, it, Y, e, nitems
    if (int8_tile) {
        switch (cls) {
        case 0: launch<16, int8_t>(QB_ARGS); return true;
        case 1: launch<8, int8_t>(QB_ARGS); return true;
        case 2: launch<4, int8_t>(QB_ARGS); return true;
        case 3: launch<2, int8_t>(QB_ARGS); return true;
        case 4: launch<1, int8_t>(QB_ARGS); return true;
        }
    } else {
        switch (cls) {
        case 1: launch<8, int16_t>(QB_ARGS); return true;
        case 2: launch<4, int16_t>(QB_ARGS); return true;
        case 3: launch<2, int16_t>(QB_ARGS); return true;
        case 4: launch<1, int16_t>(QB_ARGS); return true;
        }
    }
#undef QB_ARGS
    return false;
}
