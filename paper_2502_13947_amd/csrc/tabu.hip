// Tabu search (Alg. 1 of the IC-D^2S paper) on gfx950: one workgroup per
// solution, of one wave up to 1536 variables, four up to 8192 and eight
// beyond (qb_tabu_threads).
//
// Thread t owns the variables j = e*TB + t (e < EPT) and keeps in
// registers, per variable: a key of the move value D_j = Q_jj + 2(1-2x_j)h_j
// (biased to be non-negative), the element e and, in the top bit, whether the
// variable is tabu; and the factor S_j = 2(1-2x_j).
//
// One step: every lane takes the minimum of its allowed keys (not tabu, or
// aspirating: OV + D < OV_min); the wave minimum comes from DPP row
// operations and the row broadcasts; index order inside a wave is (element,
// lane), so the lowest lane holding the minimal key gives the lowest index;
// the wave winners meet in LDS (one barrier per step, double-buffered slots,
// the step loop run in pairs so every slot address is fixed), where a DPP
// minimum over lanes picks the smallest (32-bit (key, wave) when the move
// values allow, else 64-bit (move, index, x)).  The chosen variable's row is
// read from the Tabu copy of Q, where each thread's elements lie in one
// padded, naturally aligned slot of up to 16 bytes, or in a few aligned
// chunks beyond that (qb_tabu_pos); each element's update is one dot product
// of its row word with S_j at the element's place of the word.  x_min is
// never copied: per-variable "flipped since the last improvement" bits
// recover it, and the field is moved to x_min with the rows of the differing
// variables.
//
// What bounds it: the instructions of one step's chain, which every wave
// walks (without the row loads a step takes as long, so memory is hidden).
// Hence few waves, no per-element work but a dot product and two minima, and
// everything that is not on the way from a row to the next winner -- the
// owner's patch, the tabu lists, the books -- placed while the row is on its
// way.  One variable at most is released per step without any scan: the ring
// of flips names it.  Against sixteen waves that scanned their own release
// steps and patched after the row: n = 7000, 256 solutions 0.99 -> 0.70 us
// per step, n = 2500 0.75 -> 0.58, n = 1000 0.63 -> 0.50, n = 256 0.60 -> 0.46.
#include <algorithm>

#include "qb_internal.h"

#include <type_traits>

namespace {

// Cross-wave winner in 32 bits (K32): the slot's low word is
// (wave minimum key << WB) | wave and its high word (lane << 1) | x, with
// NW = TB / 64 waves and WB = log2 NW.  Within a wave the ballot already
// took the lowest lane among equal keys, and across waves (move, element,
// wave) orders exactly as (move, index) since index = element * TB + wave *
// 64 + lane; so a 32-bit DPP minimum over the slots picks the winner and one
// readlane of the winning slot's high word gives its lane and x.  Used when
// every real key fits 31 - WB bits.
template <int TB>
struct TabuShape {
    static constexpr int NW = TB / 64;
    static constexpr int WB = qb_ceil_log2(NW);
    static_assert(NW <= 16 && (NW & (NW - 1)) == 0, "a power of two of waves");
};

constexpr int qb_pow2_at_least(int v) { return v <= 1 ? 1 : 2 * qb_pow2_at_least((v + 1) / 2); }

// A thread's elements of one row of the Tabu copy of Q (the order of
// qb_tabu_pos), as they lie in memory: element e in word e / EPW, at bit
// BITS * (e % EPW).  Up to 16 bytes one naturally aligned load of the
// thread's padded slot; beyond, one load per chunk.
template <typename QT, int EPT, int TB>
struct TabuRow {
    static constexpr int ESZ = (int)sizeof(QT), EPW = 4 / ESZ, BITS = 8 * ESZ;
    static constexpr int BYTES = EPT * ESZ;
    static constexpr int SLOT = BYTES <= 16 ? qb_pow2_at_least(BYTES) : BYTES;
    static_assert(SLOT <= 16 || SLOT % 4 == 0, "whole words");
    static constexpr int NWD = (SLOT + 3) / 4;
    uint32_t w[NWD];

    // the chunk of SZ bytes at byte START of the thread's part, then the rest;
    // the row's byte offset is a scalar, the thread's an unchanging register
    template <int START = 0, int SZ = 16>
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rows, uint32_t row, uint32_t tid)
    {
        if constexpr (START < SLOT) {
            if constexpr (SLOT - START >= SZ) {
                const uint32_t at = START * TB + tid * (uint32_t)SZ;
                if constexpr (SZ == 16) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rows, at, row, 0);
#pragma unroll
                    for (int k = 0; k < 4; ++k) w[START / 4 + k] = v[k];
                } else if constexpr (SZ == 8) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b64(rows, at, row, 0);
                    w[START / 4] = v[0]; w[START / 4 + 1] = v[1];
                } else if constexpr (SZ == 4) {
                    w[START / 4] = __builtin_amdgcn_raw_buffer_load_b32(rows, at, row, 0);
                } else if constexpr (SZ == 2) {
                    w[START / 4] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rows, at, row, 0);
                } else {
                    w[START / 4] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rows, at, row, 0);
                }
                load<START + SZ, SZ>(rows, row, tid);
            } else {
                load<START, SZ / 2>(rows, row, tid);
            }
        }
    }

    // a factor at element e's place of its word, and c + factor * element e:
    // one dot product of the word with the factor's word (the other places 0)
    static __device__ __forceinline__ uint32_t place(int e, int32_t f)
    {
        return ((uint32_t)f & (BITS == 8 ? 0xFFu : 0xFFFFu)) << (BITS * (e % EPW));
    }
    __device__ __forceinline__ uint32_t mad(int e, uint32_t factor, uint32_t c) const
    {
        if constexpr (ESZ == 1) {
            return (uint32_t)__builtin_amdgcn_sdot4((int)w[e / EPW], (int)factor, (int)c, false);
        } else {
            typedef short v2s __attribute__((ext_vector_type(2)));
            return (uint32_t)__builtin_amdgcn_sdot2(__builtin_bit_cast(v2s, w[e / EPW]),
                                                    __builtin_bit_cast(v2s, factor), (int)c, false);
        }
    }
};

// The words of a row are not looked at before this point.
template <int N>
__device__ __forceinline__ void tabu_arrive(uint32_t (&w)[N])
{
#pragma unroll
    for (int k = 0; k < N; ++k) asm volatile("" : "+v"(w[k]));
}

// A value computed in every lane (an update under a condition would copy the
// whole vector around a branch).
__device__ __forceinline__ uint32_t tabu_held(uint32_t v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// *p += 1 in LDS, nothing returned.
__device__ __forceinline__ void lds_inc(int32_t *p)
{
    const uint32_t a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int32_t *)p;
    asm volatile("ds_add_u32 %0, %1" ::"v"(a), "v"(1) : "memory");
}

// A flip in the ring: beyond 8192 variables two bytes, for more of them.
template <int TB>
using TabuFlip = std::conditional_t<(TB > 256), uint16_t, int32_t>;

template <int EPT, typename QT, bool K32, int TB>
__global__ void __launch_bounds__(TB) k_tabu(const QT *__restrict__ Qt, int ldp, const int32_t *__restrict__ diag,
                                             int n, uint8_t *__restrict__ X, int32_t *__restrict__ H,
                                             int64_t *__restrict__ E, int alpha, int tenure, int asp,
                                             int32_t *__restrict__ Tout, int32_t *__restrict__ LFout,
                                             uint32_t bias, int ring)
{
    constexpr int NW = TabuShape<TB>::NW, WB = TabuShape<TB>::WB;
    constexpr int EB = qb_ceil_log2(EPT);           // bits of the element index
    constexpr uint32_t EMASK = (1u << EB) - 1u;
    __shared__ uint64_t red[2][NW];
    __shared__ uint64_t red2[NW];
    __shared__ int32_t list[TB + 3];             // padded to a multiple of 4 with 0 = no row
    __shared__ int lcount;
    extern __shared__ int32_t tl[];              // the ring; [n] flips, [n] last-flip steps
    TabuFlip<TB> *hist = reinterpret_cast<TabuFlip<TB> *>(tl);
    int32_t *Ts = tl + ring * (int)sizeof(TabuFlip<TB>) / 4, *Ls = Ts + n;

    const int p = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t ro = (int64_t)p * n;
    constexpr uint32_t TBIT = 0x80000000u;       // set in a key while the variable is tabu
    constexpr uint32_t KNONE = 0xFFFFFFFFu;
    // padding elements carry the largest possible key, tabu for ever
    const uint32_t dpad = 0x7FFFFFFFu >> EB;

    using Row = TabuRow<QT, EPT, TB>;
    const uint32_t pitch = (uint32_t)ldp * (uint32_t)sizeof(QT);
    // n * pitch stays below 2^30 bytes; 0x27000: raw 32-bit elements
    const __amdgpu_buffer_rsrc_t rows =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<QT *>(Qt), 0, (uint32_t)n * pitch, 0x27000);
    // a row's product with S_j changes sign with the flip's direction: the
    // bits in which +S and -S differ, at each place of a word
    constexpr int32_t S0 = 2 << EB;
    constexpr uint32_t SX = ((uint32_t)S0 ^ (uint32_t)-S0) & (Row::BITS == 8 ? 0xFFu : 0xFFFFu);
    static_assert(S0 < 128, "S fits a byte");

    // vectors, not arrays: a uniform index into sixteen or more elements moves
    // one register (a select per element below that)
    constexpr int KW = EPT <= 2 ? EPT : EPT <= 16 ? 16 : 32;
    typedef uint32_t Keys __attribute__((ext_vector_type(KW)));
    Keys Kb;               // ((D + bias) << EB | e) | TBIT if tabu
    Keys S;                // turned * 2 (1 - 2 x) << EB, at the element's place of a row word
    uint32_t xb = 0;       // x bits of the owned variables (EPT <= 32)
    uint32_t pb = 0;       // flipped since the last improvement
    uint32_t late = 0;     // variables whose release the thread looks up itself
    int32_t nexp = 0x7fffffff;   // the last tabu step of the first of those
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int j = e * TB + tid;
        if (j < n) {
            const int32_t x = X[ro + j] & 1;
            const int32_t qjj = diag[j];
            S[e] = Row::place(e, x ? -S0 : S0);
            xb |= (uint32_t)x << e;
            Kb[e] = (((uint32_t)(qjj + (x ? -2 : 2) * H[ro + j]) + bias) << EB) | (uint32_t)e;
            Ts[j] = 0;
            Ls[j] = 0;
        } else {
            S[e] = 0;
            Kb[e] = (dpad << EB) | (uint32_t)e | TBIT;   // never released
        }
    }
    int64_t OVmin = E[p];
    int64_t gap = 0;       // OV - OV_min, never negative
    int32_t turned = 1;    // the direction of the last flip
    const int wu = __builtin_amdgcn_readfirstlane(wid);
    // A variable flipped at step t is tabu through step t + tenure - 1, plus
    // the tenure that was left when it aspirated.  Without such a rest the
    // ring of flips names it when its time is over (all ones: nobody).  With
    // one, or with a tenure past the ring, it is `late`: its last tabu step
    // waits in Tout (scratch until the end) and nexp.  A tenure that reaches
    // the last step releases nobody.
    const int rmask = ring - 1;
    const bool never = tenure >= alpha;
    const uint32_t vend = never ? 0u : 0xFFFFu;   // the ring releases variables below
    const uint32_t far = !never && tenure >= ring;
    const uint32_t tnew = tenure >= 2 ? TBIT : 0u;
    for (int t = tid; t < ring; t += TB) hist[t] = (TabuFlip<TB>)-1;
    // aspiration: a tabu key k aspirates when (k >> EB) < OV_min - OV + bias,
    // that is k < tbk (zero when nothing can aspirate)
    uint32_t tbk = asp ? bias << EB : 0u;

    // One step; consecutive steps alternate the two slot buffers, so the loop
    // runs in pairs and every LDS address is fixed.
    auto one_step = [&](const int step, uint64_t *slots) {
        // smallest free key (tabu keys carry bit 31, so they lose the
        // unsigned minimum) and smallest tabu key (they win the signed one);
        // the smallest tabu key aspirates whenever any does
        uint32_t m1 = KNONE;
        int32_t m2 = 0x7fffffff;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            m1 = min(m1, Kb[e]);
            m2 = min(m2, (int32_t)Kb[e]);
        }
        const uint32_t fk = (uint32_t)max((int32_t)m1, -1);    // KNONE when every key is tabu
        const uint32_t tk = (uint32_t)m2 ^ TBIT;               // >= TBIT (never aspirates) when none is
        const uint32_t best = min(fk, tk < tbk ? tk : KNONE);
        // a lane's half of its wave's winner slot, should it win: its number
        // and its best variable's x
        auto mark_of = [&](uint32_t bsel) { return (uint32_t)lane << 1 | ((xb >> (bsel & EMASK)) & 1u); };
        const uint32_t mark = mark_of(best);
        const uint32_t wmin = qb_wave_min_u32_b(best);
        // lowest index among the minimal moves of the wave: the lowest lane
        // holding the minimal key (move, element)
        auto lane_of = [&](uint32_t wm, uint32_t bsel) { return (int)__builtin_ctzll(__ballot(bsel == wm)); };
        // the wave's winner slot for minimum key wm among the lanes' keys bsel
        // (a whole-wave call); padding keys, and no key at all, never win a
        // K32 slot
        auto slot_of = [&](uint32_t wm, uint32_t bsel, uint32_t mark) -> uint64_t {
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)mark, lane_of(wm, bsel));
            if constexpr (K32)
                return ((uint64_t)hi << 32) | (wm >= (1u << (31 - WB)) ? ~0u : (wm << WB) | (uint32_t)wu);
            else
                return wm == KNONE ? ~0ull
                                   : qb_tabu_winner(wm >> EB, (int)(wm & EMASK) * TB + wu * 64 + (int)(hi >> 1), hi & 1u);
        };
        uint32_t dib;
        int i, ei, ti;                             // the variable, its element and thread
        int32_t s;                                 // direction of x_i
        if constexpr (NW == 1) {
            __builtin_amdgcn_wave_barrier();
            uint32_t wm = wmin, bsel = best;
            if (__builtin_expect(wm == KNONE, 0)) {
                // every variable is tabu and none aspirates: argmin over all of them
                bsel = min(fk, tk);
                wm = qb_wave_min_u32_b(bsel);
            }
            ti = lane_of(wm, bsel);
            dib = wm >> EB;
            ei = (int)(wm & EMASK);
            s = ((uint32_t)__builtin_amdgcn_readlane((int)xb, ti) >> ei) & 1u ? -1 : 1;
            i = ei * TB + ti;
        } else {
            const uint64_t wkey = slot_of(wmin, best, mark);
            if (lane == 0) slots[wid] = wkey;
            qb_lds_barrier();
            if constexpr (K32) {
                uint32_t key, hi;
                if (__builtin_expect(!qb_pick32<NW>(slots, lane, key, hi), 0)) {
                    // every variable is tabu and none aspirates: argmin over all of them
                    const uint32_t b2 = min(fk, tk);
                    const uint32_t w2 = qb_wave_min_u32_b(b2);
                    const uint64_t k2 = slot_of(w2, b2, mark_of(b2));
                    if (lane == 0) red2[wid] = k2;
                    qb_lds_barrier();
                    qb_pick32<NW>(red2, lane, key, hi);
                }
                const uint32_t wm = key >> WB;
                dib = wm >> EB;
                ei = (int)(wm & EMASK);
                ti = (int)(key & (NW - 1)) * 64 + (int)(hi >> 1);
                i = ei * TB + ti;
                s = (hi & 1u) ? -1 : 1;
            } else {
                uint64_t kb = qb_min_winners<NW>(slots, lane);
                if (__builtin_expect(kb == ~0ull, 0)) {
                    // every variable is tabu and none aspirates: argmin over all of them
                    const uint32_t b2 = min(fk, tk);
                    const uint32_t w2 = qb_wave_min_u32_b(b2);
                    const uint64_t k2 = slot_of(w2, b2, mark_of(b2));
                    if (lane == 0) red2[wid] = k2;
                    qb_lds_barrier();
                    kb = qb_min_winners<NW>(red2, lane);
                }
                dib = (uint32_t)(kb >> 32);
                i = (int)((uint32_t)kb >> 1);
                ti = i & (TB - 1);
                ei = i / TB;
                s = (kb & 1) ? -1 : 1;
            }
        }
        // the row base is uniform (scalar registers); each lane adds its own
        // 32-bit chunk offsets
        Row q;
        q.load(rows, (uint32_t)i * pitch, (uint32_t)tid);

        // Everything else of the step while the row is on its way.
        const uint32_t rel = (uint32_t)hist[(step - tenure + 1) & rmask];
        gap += (int32_t)(dib - bias);
        if ((ti >> 6) == wu) {
            // the owner patches its element: minus the old move value (the
            // row's diagonal is zero in the Tabu copy, so the update below
            // leaves it)
            const bool mine = lane == (ti & 63);
            const uint32_t old = Kb[ei], sgn = S[ei];
            Kb[ei] = tabu_held(mine ? ((2u * bias - dib) << EB) | (uint32_t)ei | tnew : old);
            S[ei] = tabu_held(sgn ^ (mine ? SX << (Row::BITS * (ei % Row::EPW)) : 0u));
            const uint32_t bit = mine ? 1u << ei : 0u;
            xb ^= bit;
            pb ^= bit;
            if (__builtin_expect(far | (__ballot((int32_t)old < 0) >> (ti & 63) & 1u), 0)) {
                if (mine && tnew && !never) {
                    int32_t left = 0;
                    if (old & TBIT) {
                        const int64_t u = (late >> ei) & 1u ? (int64_t)Tout[ro + i] : (int64_t)Ls[i] + tenure - 1;
                        left = max((int32_t)min(u, (int64_t)alpha + 1) - (step - 1), 0);
                    }
                    // alpha + 1 is past the last step
                    const int32_t un = (int32_t)min((int64_t)step + left + tenure - 1, (int64_t)alpha + 1);
                    Tout[ro + i] = un;
                    late |= 1u << ei;
                    nexp = min(nexp, un);
                }
            }
            if (mine) Ls[i] = step;
        }
        // the books by another wave than the owner's
        if (((ti >> 6) + NW / 2) % NW == wu && lane == 0) {
            lds_inc(&Ts[i]);
            hist[step & rmask] = (TabuFlip<TB>)i;
        }
        {
            // the variable that is free again at the next step
            const int v = __builtin_amdgcn_readfirstlane((int)rel);
            if ((uint32_t)v < vend && ((v >> 6) & (NW - 1)) == wu) {
                const int ev = v / TB;
                const uint32_t kv = Kb[ev];
                Kb[ev] = tabu_held(lane == (v & 63) && !((late >> ev) & 1u) ? kv & ~TBIT : kv);
            }
        }
        if (__builtin_expect(__ballot(step >= nexp) != 0, 0)) {
            // the elements that are late in any lane, four at a time: their
            // steps are read together (n = 7000, a step in the mean: 0.68 us,
            // 0.70 with every element looked at in turn, 0.72 with the lanes'
            // masks shuffled together)
            nexp = 0x7fffffff;
            uint32_t any = 0;
#pragma unroll
            for (int e = 0; e < EPT; ++e) any |= __ballot((late >> e) & 1u) ? 1u << e : 0u;
#pragma unroll 1
            while (any) {
                int el[4], u[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    el[k] = any ? __builtin_ctz(any) : EPT;
                    any &= any - 1;
                    u[k] = el[k] < EPT && (late >> el[k]) & 1u ? Tout[ro + el[k] * TB + tid] : 0x7fffffff;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (el[k] >= EPT) break;
                    const uint32_t kv = Kb[el[k]];
                    Kb[el[k]] = tabu_held(u[k] <= step ? kv & ~TBIT : kv);
                    late &= u[k] <= step ? ~(1u << el[k]) : ~0u;
                    nexp = min(nexp, u[k] <= step ? 0x7fffffff : u[k]);
                }
            }
        }
        if ((int32_t)((uint64_t)gap >> 32) < 0) {
            // a new best: x_min is the current x
            OVmin += gap;
            gap = 0;
            pb = 0;
        }
        tbk = asp && (uint64_t)gap < bias ? (bias - (uint32_t)gap) << EB : 0u;
        // ready before the row is (one wave alone does better with the
        // compiler's order)
        if constexpr (NW > 1) asm volatile("" : "+s"(tbk));
        // the signs follow the flip's direction
        if (s != turned) {
            turned = s;
#pragma unroll
            for (int e = 0; e < EPT; ++e) S[e] ^= SX << (Row::BITS * (e % Row::EPW));
        }

        // h_j += s Q_ji  =>  D_j += S_j s Q_ji, applied to the key above its
        // element bits
        tabu_arrive(q.w);
#pragma unroll
        for (int e = 0; e < EPT; ++e) Kb[e] = q.mad(e, S[e], Kb[e]);
    };

    int step = 1;
    for (; step < alpha; step += 2) {
        one_step(step, red[1]);
        one_step(step + 1, red[0]);
    }
    if (step == alpha) one_step(step, red[1]);

    // field of the final x from D, then moved to x_min = x ^ pb row by row
    int32_t h[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int j = e * TB + tid;
        h[e] = 0;
        if (j < n) {
            const int32_t qjj = diag[j];
            h[e] = ((int32_t)(((Kb[e] & ~TBIT) >> EB) - bias) - qjj) * (((xb >> e) & 1u) ? -2 : 2) / 4;
            // the diagonal's part of the move to x_min (zero in the Tabu copy)
            if ((pb >> e) & 1u) h[e] += ((xb >> e) & 1u) ? -qjj : qjj;
        }
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        if (tid == 0) lcount = 0;
        __syncthreads();
        if (e * TB + tid < n && ((pb >> e) & 1u)) {
            const int pos = atomicAdd(&lcount, 1);
            const int jj = e * TB + tid;
            list[pos] = ((xb >> e) & 1u) ? -(jj + 1) : (jj + 1);
        }
        __syncthreads();
        const int cnt = lcount;
        if (tid < 3) list[cnt + tid] = 0;
        __syncthreads();
        for (int u = 0; u < cnt; u += 4) {           // four rows on their way at once
            Row q[4];
            int32_t sg[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int32_t v = __builtin_amdgcn_readfirstlane(list[u + k]);
                sg[k] = v > 0 ? 1 : v < 0 ? -1 : 0;
                q[k].load(rows, (uint32_t)(v > 0 ? v - 1 : v < 0 ? -v - 1 : 0) * pitch, (uint32_t)tid);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e2 = 0; e2 < EPT; ++e2) h[e2] = (int32_t)q[k].mad(e2, Row::place(e2, sg[k]), (uint32_t)h[e2]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int j = e * TB + tid;
        if (j < n) {
            X[ro + j] = (uint8_t)(((xb ^ pb) >> e) & 1u);
            H[ro + j] = h[e];
            Tout[ro + j] = Ts[j];
            LFout[ro + j] = Ls[j];
        }
    }
    if (tid == 0) E[p] = OVmin;
}

template <int EPT, typename QT, bool K32, int TB>
qb_status launch_one(const QT *Qt, int ldp, qb_problem P, int z, uint8_t *X, int32_t *H, int64_t *E, int alpha,
                     int tenure, int asp, int32_t *T, int32_t *LF, uint32_t bias, hipStream_t s)
{
    // The ring holds the tenure's flips (a power of two of them, 1024 or
    // more) as far as LDS has room: every tenure up to n below 15,600
    // variables, 8191 beyond.  Past it each release is looked up: n = 7000,
    // tenure 1024, 0.76 us a step with a ring of 2048 and 3.6 with 1024
    // (n / 150: 0.70); n = 16384, tenure 5000, 0.88 and 3.2.
    constexpr int LDS_MAX = 160 * 1024, fixed = 24 * TabuShape<TB>::NW + 4 * (TB + 4) + 64;   // static arrays
    constexpr int flip = (int)sizeof(TabuFlip<TB>);
    const int room = LDS_MAX - fixed - 8 * P->n;
    int ring = 1024;
    if (tenure < alpha)
        while (ring <= tenure && 2 * ring * flip <= room) ring *= 2;
    const int lds = 8 * P->n + ring * flip;
    QB_TRY_HIP(hipFuncSetAttribute((const void *)k_tabu<EPT, QT, K32, TB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   lds));
    k_tabu<EPT, QT, K32, TB><<<z, TB, lds, s>>>(Qt, ldp, P->diag, P->n, X, H, E, alpha, tenure, asp, T, LF, bias, ring);
    QB_LAUNCH_CHECK();
    return QB_OK;
}

// The 32-bit winner key when every real key fits 31 - WB bits, else 64 bits.
template <int EPT, typename QT, int TB>
qb_status launch_keyed(const QT *Qt, int ldp, qb_problem P, int z, uint8_t *X, int32_t *H, int64_t *E,
                       int alpha, int tenure, int asp, int32_t *T, int32_t *LF, int64_t dmax, hipStream_t s)
{
    if (2 * dmax + 1 >= (int64_t)(0x7FFFFFFFu >> qb_ceil_log2(EPT))) return QB_E_RANGE;
    const uint32_t bias = (uint32_t)dmax;
    // one wave has no winners to compare, and int8 moves always fit
    // (2 dmax + 1 <= 254 (2 n + 1) + 1 < 2^23 for n = 16384)
    constexpr bool always = TB == 64 || (sizeof(QT) == 1 && TB < QB_TABU_THREADS);
    if (TB < QB_TABU_THREADS && ((2 * dmax + 1) << qb_ceil_log2(EPT)) < (int64_t(1) << (31 - TabuShape<TB>::WB)))
        return launch_one<EPT, QT, (TB < QB_TABU_THREADS), TB>(Qt, ldp, P, z, X, H, E, alpha, tenure, asp, T, LF, bias,
                                                              s);
    return launch_one<EPT, QT, always, TB>(Qt, ldp, P, z, X, H, E, alpha, tenure, asp, T, LF, bias, s);
}

template <typename QT>
qb_status launch_tabu(qb_problem P, const QT *Qt, int ldp, int z, uint8_t *X, int32_t *H, int64_t *E, int alpha,
                      int tenure, int asp, int32_t *T, int32_t *LF, hipStream_t s)
{
    const int ept = P->tabu_ept, tb = P->tabu_tb;
    if (ept == 0 || ldp != qb_tabu_pitch(tb, ept, (int)sizeof(QT))) return QB_E_CAPACITY;
    const int64_t dmax = (int64_t)P->qmax + 2 * P->eta_max;
#define QB_T(K, W)                                                                                 \
    if (ept == K && tb == W)                                                                      \
        return launch_keyed<K, QT, W>(Qt, ldp, P, z, X, H, E, alpha, tenure, asp, T, LF, dmax, s);
    QB_T(1, 64) QB_T(2, 64) QB_T(4, 64) QB_T(6, 64) QB_T(8, 64) QB_T(10, 64) QB_T(12, 64) QB_T(14, 64)
    QB_T(16, 64) QB_T(20, 64) QB_T(24, 64)
    QB_T(8, 256) QB_T(10, 256) QB_T(12, 256) QB_T(14, 256) QB_T(16, 256) QB_T(20, 256) QB_T(24, 256)
    QB_T(28, 256) QB_T(32, 256)
    QB_T(20, 512) QB_T(24, 512) QB_T(28, 512) QB_T(32, 512)
    // move values past the others' keys: 16-bit weights only
    if constexpr (sizeof(QT) == 2) {
        QB_T(1, 1024) QB_T(2, 1024) QB_T(3, 1024) QB_T(4, 1024) QB_T(5, 1024) QB_T(6, 1024)
        QB_T(7, 1024) QB_T(8, 1024) QB_T(10, 1024) QB_T(12, 1024) QB_T(14, 1024) QB_T(16, 1024)
    }
#undef QB_T
    return QB_E_CAPACITY;
}

}  // namespace

qb_status qb_tabu_sparse_launch(qb_problem P, int z, uint8_t *X, int32_t *H, int64_t *E, int alpha, int tenure,
                                int asp, int32_t *T, int32_t *LF, hipStream_t s);

extern "C" qb_status qb_tabu(qb_problem P, int32_t z, uint8_t *X_d, int32_t *H_d, int64_t *E_d,
                            int32_t alpha, int32_t tenure, int32_t aspiration, int32_t *T_d,
                            int32_t *LF_d, void *stream)
{
    if (!P || z < 1 || !X_d || !H_d || !E_d || !T_d || !LF_d || alpha < 0 || tenure < 0)
        return QB_E_ARG;
    // a tenure that reaches past the last step keeps a variable tabu to the
    // end either way: alpha + 1 gives the same search and keeps the kernels'
    // step and counter arithmetic far from int32 overflow
    tenure = (int32_t)std::min<int64_t>(tenure, (int64_t)alpha + 1);
    hipStream_t s = qb_stream(stream);
    if (P->sparse)
        return qb_tabu_sparse_launch(P, z, X_d, H_d, E_d, alpha, tenure, aspiration != 0, T_d, LF_d, s);
    if (P->tabu_ept == 0) return QB_E_CAPACITY;
    if (P->int8_ok)
        return launch_tabu<int8_t>(P, (const int8_t *)P->Qt, P->ldp, z, X_d, H_d, E_d, alpha, tenure,
                                   aspiration != 0, T_d, LF_d, s);
    return launch_tabu<int16_t>(P, (const int16_t *)P->Qt, P->ldp, z, X_d, H_d, E_d, alpha, tenure,
                                aspiration != 0, T_d, LF_d, s);
}
