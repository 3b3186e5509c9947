// Sparse sub-QUBOs: extraction into a per-job ELL (eq. 4, sub-QUBO
// construction in Alg. 3) and the batched Ising-machine stage of Alg. 3 on it,
// on gfx950.
//
// The annealer takes the dense kernel's random numbers and thresholds, so Y
// and e are bit-identical to it: lane L owns positions 64*s + L.  What
// differs is where the fields live and how an accept updates them.  Row k of
// a sparse tile has a handful of entries, so instead of every lane adding its
// slice of a dense row, the flip bases F of each replica live in LDS and an
// accepted row's entries are added there by LDS atomic adds.  The job's ELL
// tile is staged in LDS once and shared by the rw replicas (waves) of the
// workgroup; rw only changes the schedule.
#include <algorithm>

#include "qb_internal.h"

namespace {

constexpr int DBLK_BYTES = 64 * 64;   // one diagonal block, int8

// ------------------------------------------------------------------ extract
// One workgroup per job, one thread per row: the entries of Q's row S_a whose
// column is in S become the row's ELL words with local column indices; c and
// F0 as in the dense extraction.  Rows are read and written 16 bytes at a
// time.  TABLE: a variable's place in S is looked up in an LDS table over all
// n variables, else searched for in S (qb_extract_ell says when).
template <bool TABLE>
__global__ void __launch_bounds__(1024) k_extract_ell(const uint32_t *__restrict__ ell, int W,
                                                      const int32_t *__restrict__ ecnt,
                                                      const int32_t *__restrict__ diag, int n,
                                                      const int32_t *__restrict__ sol,
                                                      const int32_t *__restrict__ off,
                                                      const int32_t *__restrict__ idx,
                                                      const uint8_t *__restrict__ X,
                                                      const int32_t *__restrict__ H, uint32_t *__restrict__ tiles,
                                                      int32_t *__restrict__ c, int32_t *__restrict__ F0,
                                                      uint8_t *__restrict__ y0, uint8_t *__restrict__ dblk,
                                                      const int32_t *__restrict__ dboff)
{
    // TABLE: [n] 1 + place in S, with x in bit 15; 0 outside.  Else [m]
    // twice the variable plus x, ascending
    extern __shared__ __align__(16) uint32_t lds[];
    uint16_t *place = reinterpret_cast<uint16_t *>(lds);
    const int q = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const int base = off[q], m = off[q + 1] - base, p = sol[q];
    const int64_t xo = (int64_t)p * n;
    if constexpr (TABLE) {
        for (int t = tid; t < (n + 7) / 8; t += nt) reinterpret_cast<uint4 *>(place)[t] = make_uint4(0, 0, 0, 0);
    }
    // the job's diagonal 64 x 64 blocks (int8), zeroed before the rows fill them
    uint8_t *dq = dblk ? dblk + (size_t)dboff[q] * DBLK_BYTES : nullptr;
    if (dq) {
        const int n16 = qb_tile_ms(m) * DBLK_BYTES / 16;
        for (int t = tid; t < n16; t += nt) reinterpret_cast<uint4 *>(dq)[t] = make_uint4(0, 0, 0, 0);
    }
    if constexpr (TABLE) __syncthreads();
    const int a = tid;                                   // m <= the workgroup's threads: a row per thread
    int i = 0;
    int32_t y = 0;
    if (a < m) {
        i = idx[base + a];
        y = X[xo + i];
        if constexpr (TABLE)
            place[i] = (uint16_t)(1 + a + (y ? 0x8000 : 0));
        else
            lds[a] = 2u * (uint32_t)i + (y ? 1u : 0u);
    }
    __syncthreads();
    if (a >= m) return;
    // 1 + place in S, with x in bit 15, of a variable; 0 outside
    auto find = [&](int j) -> uint32_t {
        if constexpr (TABLE) {
            return place[j];
        } else {
            int lo = 0;                                  // the last place whose variable is at most j
            for (int h = m; h > 1;) {
                const int half = h >> 1;
                lo = lds[lo + half] < 2u * (uint32_t)j + 2u ? lo + half : lo;
                h -= half;
            }
            const uint32_t v = lds[lo];
            return v >> 1 == (uint32_t)j ? 1u + (uint32_t)lo + ((v & 1u) << 15) : 0u;
        }
    };
    const int32_t qii = diag[i];
    const int32_t f0 = qii + 2 * (H[xo + i] - qii * y);
    F0[base + a] = f0;
    y0[base + a] = (uint8_t)y;
    const uint4 *row = reinterpret_cast<const uint4 *>(ell + (int64_t)i * W);
    uint4 *out = reinterpret_cast<uint4 *>(tiles + (int64_t)(base + a) * W);
    const int cnt = ecnt[i];
    int k = 0;
    int32_t rowsum = 0;
    uint32_t o[4] = {0u, 0u, 0u, 0u};
    for (int t = 0; t < cnt; t += 4) {
        const uint4 v4 = row[t >> 2];
        const uint32_t wv[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (t + u >= cnt) break;
            const uint32_t pl = find(qb_ell_col(wv[u]));
            if (pl == 0u) continue;
            const int32_t v = qb_ell_val(wv[u]);
            const int pos = (int)(pl & 0x7fffu) - 1;
            const uint32_t word = qb_ell_word(v, pos);
            rowsum += pl & 0x8000u ? v : 0;
            const int s = k & 3;
            o[0] = s == 0 ? word : o[0];
            o[1] = s == 1 ? word : o[1];
            o[2] = s == 2 ? word : o[2];
            o[3] = s == 3 ? word : o[3];
            if (s == 3) {
                out[k >> 2] = make_uint4(o[0], o[1], o[2], o[3]);
                o[0] = o[1] = o[2] = o[3] = 0u;
            }
            ++k;
            // column a & 63 of the block holds T[b][a] for the rows b of a's block
            if (dq && (pos >> 6) == (a >> 6))
                dq[(size_t)(a >> 6) * DBLK_BYTES + (a & 63) * 64 + (pos & 63)] = (uint8_t)(int8_t)v;
        }
    }
    // the started group, then the padding (zero words)
    for (int g = k >> 2; g < W / 4; ++g) {
        out[g] = make_uint4(o[0], o[1], o[2], o[3]);
        o[0] = o[1] = o[2] = o[3] = 0u;
    }
    if (c) c[base + a] = f0 - 2 * rowsum;
}

// ------------------------------------------------------------------ anneal
// One wave per replica, lane L holding the positions 64 s + L; F lives in LDS.
// A sweep goes one of two ways, both exact, chosen by the positions that would
// accept at its start.
//
// Many: the whole sweep is decided at once and repaired until it agrees with
// the sequential one (the fixed point of evaluating every position against a
// guess of all decisions is the sequential sweep's, as a position's answer
// depends on lower positions only).  A row of a sparse tile reaches few
// positions, so almost every first guess is right: on the sub-QUBOs of the
// n = 20000 workload (1024 variables, 230 accepts a sweep) 2.8 rounds change
// anything.  A round compares every position's field with its threshold and
// adds what the changed decisions make of the fields of *later* positions (LDS
// atomic adds); once nothing changes, the accepted rows' entries at earlier
// positions are added too.  Entries ascend by column, so a row's earlier part
// comes first; of either part the first entry is in registers, and the others
// are read from the tile in LDS by the few lanes that have any.
//
// Few: one accept after another, a block of 64 positions at a time: the lowest
// accepting lane by ballot and find-first-set, its whole row added by all
// lanes, the block's fields read again.  A chain of accepts, but rows of any
// length cost the same, where the way above walks them entry by entry on a
// lane, in every round.
//
// The line between the two, `few`, lies where both took the same time at m =
// 64 to 1024 and d = 4 to 30 entries a row within the job: MS (0.1 + d / 40) +
// d / 2 + d^2 / 10 accepts, as lanes that hold one.
//
// With F exact at both ends of a sweep the energy of the whole run is
// 1/2 sum (y - y0) (F0 + F): no sweep sums it.  A sweep's thresholds are read
// from memory during the one before.
//
// Bound by a wave's own instructions and LDS round trips (16 replicas take as
// long as one).  A sweep of 128 jobs of 1024 x 16 replicas, ranked after a Tabu
// run on the n = 20000 workload, takes 4.3 us (30 accept by accept with the
// block's couplings in registers; 5.2 with the thresholds staged in LDS).  Cold
// jobs, R = 1: m = 64 and rows of 30 within the job, 2.5 accepts, 0.72 us (2.7
// all at once, 0.55 with couplings in registers); m = 512 and rows of 20, 21
// accepts, 4.4 us (5.6 and 3.5).
__device__ __forceinline__ int32_t sat_add(int32_t a, int32_t b) { return __builtin_elementwise_add_sat(a, b); }

template <int MS>
__global__ void __launch_bounds__(512) k_anneal_ell(const int32_t *__restrict__ jobs, int rgroups,
                                                    const int32_t *__restrict__ off, int W,
                                                    const uint32_t *__restrict__ tiles,
                                                    const int32_t *__restrict__ F0,
                                                    const uint8_t *__restrict__ y0, int nsw, int B,
                                                    const int32_t *__restrict__ thr, int R, int rw, uint32_t k0,
                                                    uint32_t k1, uint32_t inst_base, const qb_iter *__restrict__ it,
                                                    uint8_t *__restrict__ Y, int64_t *__restrict__ eout,
                                                    int32_t *__restrict__ acnt)
{
    constexpr int MP = 64 * MS;
    extern __shared__ __align__(16) uint32_t dl[];
    const int q = jobs[blockIdx.x / rgroups];
    const int rg = blockIdx.x % rgroups;
    const int base = off[q], m = off[q + 1] - base;
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = rg * rw + wid;
    const bool live = r < R;

    uint32_t *tl = dl;                                            // [MP][W]
    int32_t *Fall = reinterpret_cast<int32_t *>(dl + (size_t)MP * W);   // [rw][MP]
    int32_t *F = Fall + wid * MP;
    uint32_t *info = reinterpret_cast<uint32_t *>(Fall + rw * MP);   // [MP] entries: earlier, all
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(tiles + (int64_t)base * W);
        uint4 *dst = reinterpret_cast<uint4 *>(tl);
        const int n16 = m * W / 4;
        for (int t = tid; t < n16; t += nt) dst[t] = src[t];
    }
    __syncthreads();
    for (int a = tid; a < MP; a += nt) {
        int nu = 0, cnt = 0;
        if (a < m)
            for (int t = 0; t < W; ++t) {
                const uint32_t wd = tl[a * W + t];
                if (wd == 0u) continue;
                cnt = t + 1;
                if (qb_ell_col(wd) < a) nu = t + 1;
            }
        info[a] = (uint32_t)nu | ((uint32_t)cnt << 16);
    }
    int32_t M[MS];                          // -y
    uint32_t yb = 0, real = 0;              // y, and the positions of the job, a bit each
#pragma unroll
    for (int s = 0; s < MS; ++s) {
        const int pos = 64 * s + lane;
        real |= (uint32_t)(pos < m) << s;
        if (live) F[pos] = pos < m ? F0[base + pos] : 0;
        if (pos < m && y0[base + pos]) yb |= 1u << s;
        M[s] = (yb >> s) & 1u ? -1 : 0;
    }
    const uint32_t y00 = yb;
    __syncthreads();
    if (!live) return;   // no barrier follows

    // first entries: twice the coupling, and the byte offset of the field it
    // moves (none: zero into the position's own field)
    const uint32_t fo = (uint32_t)(reinterpret_cast<char *>(F) - reinterpret_cast<char *>(dl));
    int32_t dv[MS], uv[MS];
    uint32_t da[MS], ua[MS];
    uint32_t hd = 0, hd2 = 0, hu = 0, hu2 = 0;   // positions with one, and with more, later or earlier entries
    int32_t nlater = 0;
#pragma unroll
    for (int s = 0; s < MS; ++s) {
        const int pos = 64 * s + lane;
        const int nu = (int)(info[pos] & 0xFFFFu), nd = (int)(info[pos] >> 16) - nu;
        const uint32_t wu = nu > 0 ? tl[pos * W] : 0u, wd = nd > 0 ? tl[pos * W + nu] : 0u;
        uv[s] = 2 * qb_ell_val(wu);
        ua[s] = fo + 4u * (uint32_t)(nu > 0 ? qb_ell_col(wu) : pos);
        dv[s] = 2 * qb_ell_val(wd);
        da[s] = fo + 4u * (uint32_t)(nd > 0 ? qb_ell_col(wd) : pos);
        hu |= (uint32_t)(nu > 0) << s;
        hu2 |= (uint32_t)(nu > 1) << s;
        hd |= (uint32_t)(nd > 0) << s;
        hd2 |= (uint32_t)(nd > 1) << s;
        nlater += nd;
    }
    // lanes with a position that accepts, up to which the sweep takes them one by one
    const int d = 2 * __builtin_amdgcn_readfirstlane((int)qb_wave_sum_i64(nlater)) / m;
    const int a10 = MS * (1 + d / 4) + 5 * d + d * d, few = 90 * a10 / (900 + a10);
    auto field = [&](uint32_t o) { return reinterpret_cast<int32_t *>(reinterpret_cast<char *>(dl) + o); };
    // adds the first entries of the positions `who`, with the signs `neg`;
    // the other positions add zero, which takes no branch
    auto scatter = [&](uint32_t who, uint32_t neg, const int32_t (&v)[MS], const uint32_t (&at)[MS]) {
#pragma unroll
        for (int s = 0; s < MS; ++s) {
            const int32_t n = __builtin_amdgcn_sbfe((int)neg, s, 1), on = __builtin_amdgcn_sbfe((int)who, s, 1);
            atomicAdd(field(at[s]), ((v[s] ^ n) - n) & on);
        }
    };
    // adds entries from the tile, of the few lanes that have any: the earlier
    // or the later ones but for `skip`
    auto scatter_rows = [&](uint32_t who, uint32_t neg, bool later, int skip) {
        while (who) {
            const int s = __builtin_ctz(who);
            who &= who - 1;
            const int pos = 64 * s + lane;
            const int nu = (int)(info[pos] & 0xFFFFu), cnt = (int)(info[pos] >> 16);
            const int32_t f = (neg >> s) & 1u ? -2 : 2;
            const uint32_t *row = tl + pos * W;
            for (int t = (later ? nu : 0) + skip; t < (later ? cnt : nu); ++t) {
                const uint32_t wd = row[t];
                atomicAdd(F + qb_ell_col(wd), f * qb_ell_val(wd));
            }
        }
        __builtin_amdgcn_wave_barrier();                 // whole again before the next comparison
    };
    // A block's part of a sweep taken one accept after another: of its
    // candidates `on` and, once a row was added, of fields fn; the accepted
    // ones.  No lane branches: a lane without an entry adds zero to a field of
    // its own.  The next block's fields are read along after each row.
    const int wlane = min(lane, W - 1);
    auto chain_block = [&](int s, uint64_t on, int32_t ts, int32_t ys, bool &fresh, int32_t &fn) {
        const int left = m - 64 * s;
        const uint64_t block = left >= 64 ? ~0ull : (1ull << left) - 1ull;
        if (!fresh) on = __ballot((fn ^ ys) <= ts) & block;
        uint64_t am = 0;
        int kp = -1;                                     // lane of the row on its way
        uint32_t wp = 0;
        while (on) {
            const int k = __builtin_ctzll(on);
            const int32_t f = 4 * __builtin_amdgcn_readlane(ys, k) + 2;   // 2 sigma
            const uint32_t *row = tl + (64 * s + k) * W;
            if (k != kp) wp = row[wlane];
            const uint32_t wd = lane < W ? wp : 0u;
            atomicAdd(F + (wd != 0u ? qb_ell_col(wd) : lane), f * qb_ell_val(wd));
            for (int i = 64; i < W; i += 64) {
                const uint32_t v = row[min(i + lane, W - 1)];
                const uint32_t u = i + lane < W ? v : 0u;
                atomicAdd(F + (u != 0u ? qb_ell_col(u) : lane), f * qb_ell_val(u));
            }
            fresh = false;
            am |= 1ull << k;
            const int32_t fs = F[64 * s + lane];
            if (s + 1 < MS) fn = F[64 * (s + 1) + lane];
            // the next candidate's row, most often the next accept's
            on &= ~((2ull << k) - 1ull);
            kp = -1;
            if (on) {
                kp = __builtin_ctzll(on);
                wp = tl[(64 * s + kp) * W + wlane];
            }
            on = __ballot((fs ^ ys) <= ts) & block & ~((2ull << k) - 1ull);
        }
        if (am == 0 && !fresh && s + 1 < MS) fn = F[64 * (s + 1) + lane];
        return (uint32_t)__builtin_amdgcn_inverse_ballot_w64(am) << s;
    };
    // the sweep so, of the candidates `acc` at its start
    auto chain = [&](uint32_t acc, const int32_t (&tp)[MS], const int32_t (&M)[MS]) {
        uint32_t done = 0;
        bool fresh = true;                               // no row was added yet
        int32_t fn = 0;
        if constexpr (MS <= 8) {
#pragma unroll
            for (int s = 0; s < MS; ++s) {
                if (s > 0 && 64 * s >= m) break;
                asm volatile("" : "+v"(acc));            // (no block's mask ahead of its turn)
                done |= chain_block(s, __ballot((acc >> s) & 1u), tp[s], M[s], fresh, fn);
            }
        } else {
            // a loop over indexed registers: unrolled, its scalars crowd out
            // the other way's (8 % of a sweep)
            typedef int32_t Blocks __attribute__((ext_vector_type(MS)));
            Blocks t, y;
#pragma unroll
            for (int s = 0; s < MS; ++s) {
                t[s] = tp[s];
                y[s] = M[s];
            }
#pragma unroll 1
            for (int s = 0; s < MS && 64 * s < m; ++s)
                done |= chain_block(s, __ballot((acc >> s) & 1u), t[s], y[s], fresh, fn);
        }
        return done;
    };

    int32_t nacc = 0;
    const uint32_t tag = (1u << 28) | (inst_base + (it ? it->inst : 0u) + (uint32_t)q);
    constexpr int G = (MS + 3) / 4;
    const int sh = 32 - B;
    // a sweep's thresholds
    auto thresholds = [&](int sw, int32_t (&t)[MS]) {
        const int32_t *table = thr + ((size_t)sw << B);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint4 o = qb_philox(make_uint4(((uint32_t)g << 6) | (uint32_t)lane, (uint32_t)sw, (uint32_t)r, tag),
                                      k0, k1);
#pragma unroll
            for (int w = 0; w < 4; ++w)
                if (4 * g + w < MS) t[4 * g + w] = table[qb_word(o, w) >> sh];
        }
    };
    int32_t ahead[MS];
    thresholds(0, ahead);
#pragma unroll 1
    for (int sw = 0; sw < nsw; ++sw) {
        int32_t tp[MS], f0[MS];
#pragma unroll
        for (int s = 0; s < MS; ++s) f0[s] = F[64 * s + lane];
        // the next sweep's thresholds are on their way during this one
#pragma unroll
        for (int s = 0; s < MS; ++s) tp[s] = ahead[s];
        if (sw + 1 < nsw) thresholds(sw + 1, ahead);
        // dE <= t on x = F ^ -y: for y = 1, -F <= t is ~F <= t - 1 (no field
        // reaches INT32_MAX)
#pragma unroll
        for (int s = 0; s < MS; ++s) tp[s] = sat_add(tp[s], M[s]);
        auto decide = [&]() {
            uint32_t a = 0;
#pragma unroll
            for (int s = MS - 1; s >= 0; --s) a = 2 * a + (uint32_t)((F[64 * s + lane] ^ M[s]) <= tp[s]);
            return a & real;
        };
        uint32_t acc = 0;
#pragma unroll
        for (int s = MS - 1; s >= 0; --s) acc = 2 * acc + (uint32_t)((f0[s] ^ M[s]) <= tp[s]);
        acc &= real;
        const int c = __builtin_popcountll(__ballot(acc != 0u));   // lanes with a candidate
        if (c <= few) {
            if (c > 0) acc = chain(acc, tp, M);
        } else {
            scatter(acc & hd, yb, dv, da);
            scatter_rows(acc & hd2, yb, true, 1);
            while (true) {
                const uint32_t a = decide();
                const uint32_t t = (a ^ acc) & hd;
                acc = a;
                if (__ballot(t != 0u) == 0) break;
                // the other way where no longer accepted from 0, or accepted from 1
                scatter_rows(t, a ^ ~yb, true, 0);
            }
            scatter(acc & hu, yb, uv, ua);
            scatter_rows(acc & hu2, yb, false, 1);
        }
        nacc += __builtin_popcount(acc);
        yb ^= acc;
#pragma unroll
        for (int s = 0; s < MS; ++s) M[s] = -(int32_t)((yb >> s) & 1u);
    }

    uint8_t *Yr = Y + (size_t)base * R + (size_t)r * m;
    int64_t e = 0;
#pragma unroll
    for (int s = 0; s < MS; ++s) {
        const int pos = 64 * s + lane;
        if (pos < m) {
            const int y = (int)((yb >> s) & 1u), d = y - (int)((y00 >> s) & 1u);
            Yr[pos] = (uint8_t)y;
            e += (int64_t)d * ((int64_t)F0[base + pos] + F[pos]);
        }
    }
    e = qb_wave_sum_i64(e) / 2;
    const int64_t na = acnt ? qb_wave_sum_i64(nacc) : 0;
    if (lane == 0) {
        eout[(size_t)q * R + r] = e;
        if (acnt) acnt[(size_t)q * R + r] = (int32_t)na;
    }
}

constexpr size_t LDS_MAX = 160 * 1024;

// The LDS of a workgroup that the entry point admits: the job's ELL tile,
// each replica's fields, and 64 words per replica.
inline size_t ell_lds_bytes(int ms, int W, int rw)
{
    return sizeof(uint32_t) * ((size_t)64 * ms * (W + rw) + (size_t)64 * rw);
}

template <int MS>
qb_status launch_ell(int njobs, int rw, int R, hipStream_t s, const int32_t *jobs, qb_batch b, int W,
                     const uint32_t *tiles, const int32_t *F0, const uint8_t *y0, int nsw, int B, const int32_t *thr,
                     uint64_t seed, uint32_t inst_base, const qb_iter *it, uint8_t *Y, int64_t *e)
{
    // up to 8 replicas per workgroup (256 registers a lane), more in further workgroups
    rw = std::min(rw, 8);
    const int rgroups = (R + rw - 1) / rw;
    // the tile, the fields and the entry counts: no more than qb_anneal_ell_x
    // admitted, whose 64 words a replica round up to a multiple of the class
    const size_t lds = sizeof(uint32_t) * 64 * MS * (size_t)(W + rw + 1);
    if (lds > LDS_MAX) return QB_E_CAPACITY;
    // set on every launch (no cached flag shared between devices or threads)
    QB_TRY_HIP(hipFuncSetAttribute((const void *)k_anneal_ell<MS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)LDS_MAX));
    k_anneal_ell<MS><<<njobs * rgroups, 64 * rw, lds, s>>>(jobs, rgroups, b->off_d, W, tiles, F0, y0, nsw, B, thr, R,
                                                           rw, (uint32_t)seed, (uint32_t)(seed >> 32), inst_base, it,
                                                           Y, e, b->acnt_d);
    QB_LAUNCH_CHECK();
    return QB_OK;
}

qb_status dispatch_ell(int cls, int njobs, int rw, int R, hipStream_t s, const int32_t *jobs, qb_batch b, int W,
                       const uint32_t *tiles, const int32_t *F0, const uint8_t *y0, int nsw, int B,
                       const int32_t *thr, uint64_t seed, uint32_t inst_base, const qb_iter *it, uint8_t *Y, int64_t *e)
{
#define QB_ARGS njobs, rw, R, s, jobs, b, W, tiles, F0, y0, nsw, B, thr, seed, inst_base, it, Y, e
    switch (cls) {
    case 0: return launch_ell<16>(QB_ARGS);
    case 1: return launch_ell<8>(QB_ARGS);
    case 2: return launch_ell<4>(QB_ARGS);
    case 3: return launch_ell<2>(QB_ARGS);
    case 4: return launch_ell<1>(QB_ARGS);
    }
#undef QB_ARGS
    return QB_E_UNSUPPORTED;
}

}  // namespace

// `blocks`: also the int8 diagonal blocks, which no kernel reads.
qb_status qb_extract_ell_x(qb_problem P, qb_batch b, const uint8_t *X_d, const int32_t *H_d, uint32_t *tile_d,
                           int32_t *c_d, int32_t *F0_d, uint8_t *y0_d, bool blocks, void *stream)
{
    if (!P || !b || !X_d || !H_d || !tile_d || !F0_d || !y0_d) return QB_E_ARG;
    if (b->n != P->n) return QB_E_ARG;
    if (!P->sparse) return QB_E_UNSUPPORTED;
    if ((uintptr_t)tile_d & 15) return QB_E_ARG;
    if (b->J == 0) return QB_OK;
    uint8_t *dblk = blocks && P->int8_ok ? reinterpret_cast<uint8_t *>(tile_d + (int64_t)b->total * P->ellw) : nullptr;
    // The table, unless clearing it for every job costs more than searching:
    // many jobs a compute unit, of few variables and entries beside n.  20000
    // variables, rows of 40: 16384 jobs of 10 take 120 us with it and 48
    // without, of 64 160 and 120, of 128 267 and 293; 2048 jobs of 64 25 and
    // 32.  Rows of 8: 16384 jobs of 64 74 and 39, of 128 82 and 68; 247 of
    // 1024 11 and 16.  The workgroup has a row per thread, and for the table
    // at least 8 threads per KB of it.
    int ncu = 0;
    QB_TRY_HIP(qb_cu_count(&ncu));
    const bool table = (int64_t)b->J * P->n <= (int64_t)240000 * ncu || P->n <= (int64_t)b->m_max * (128 + 4 * P->ellw);
    const int nt = (std::min(std::max(b->m_max, table ? P->n / 64 : 0), 1024) + 63) / 64 * 64;
    const int lds = table ? (P->n + 7) / 8 * 16 : 4 * b->m_max;
    const auto kern = table ? k_extract_ell<true> : k_extract_ell<false>;
    QB_TRY_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    kern<<<b->J, nt, lds, qb_stream(stream)>>>(P->ell, P->ellw, P->ecnt, P->diag, P->n, b->sol_d, b->off_d, b->idx_d,
                                               X_d, H_d, tile_d, c_d, F0_d, y0_d, dblk, b->dboff_d);
    QB_LAUNCH_CHECK();
    return QB_OK;
}

extern "C" qb_status qb_extract_ell(qb_problem P, qb_batch b, const uint8_t *X_d, const int32_t *H_d,
                                   uint32_t *tile_d, int32_t *c_d, int32_t *F0_d, uint8_t *y0_d, void *stream)
{
    return qb_extract_ell_x(P, b, X_d, H_d, tile_d, c_d, F0_d, y0_d, true, stream);
}

qb_status qb_anneal_ell_x(qb_batch b, int32_t W, const uint32_t *tile_d, const int32_t *F0_d, const uint8_t *y0_d,
                          int32_t nsw, int32_t B, const int32_t *thr_d, int32_t R, int32_t rw, uint64_t seed,
                          uint32_t inst_base, const qb_iter *it, uint8_t *Y_d, int64_t *e_d, void *stream)
{
    if (!b || !tile_d || !F0_d || !y0_d || !thr_d || !Y_d || !e_d) return QB_E_ARG;
    if (nsw < 1 || B < 1 || B > 16 || R < 1 || R > 16 || rw < 0 || rw > 16) return QB_E_ARG;
    if (W < 4 || (W & 3) || W > 65536) return QB_E_ARG;
    if ((uintptr_t)tile_d & 15) return QB_E_ARG;
    if ((uint64_t)inst_base + (uint64_t)b->J > (1ull << 28)) return QB_E_RANGE;
    hipStream_t s = qb_stream(stream);
    // every size class starts at once: the fork precedes the first launch
    int ncls = 0;
    for (int c = 0; c < QB_NCLASS; ++c) ncls += b->cls_end[c] > b->cls_begin[c];
    if (ncls > 1) QB_TRY_HIP(hipEventRecord(b->ev_fork, s));
    bool first = true;
    for (int c = 0; c < QB_NCLASS; ++c) {
        const int nj = b->cls_end[c] - b->cls_begin[c];
        if (nj <= 0) continue;
        const int ms = qb_ms_of_class(c);
        int r2 = rw;
        if (r2 == 0) {
            // automatic: up to 8 replicas per workgroup, fewer when LDS is short
            r2 = R < 8 ? R : 8;
            while (r2 > 1 && ell_lds_bytes(ms, W, r2) > LDS_MAX) r2 >>= 1;
        }
        if (ell_lds_bytes(ms, W, r2) > LDS_MAX) return QB_E_CAPACITY;
        hipStream_t ls = s;
        if (!first) {
            ls = b->side[c];
            QB_TRY_HIP(hipStreamWaitEvent(ls, b->ev_fork, 0));
        }
        const qb_status rc = dispatch_ell(c, nj, r2, R, ls, b->lpt_d + b->cls_begin[c], b, W, tile_d, F0_d, y0_d, nsw,
                                          B, thr_d, seed, inst_base, it, Y_d, e_d);
        if (rc != QB_OK) return rc;
        if (!first) {
            QB_TRY_HIP(hipEventRecord(b->ev_join[c], ls));
            QB_TRY_HIP(hipStreamWaitEvent(s, b->ev_join[c], 0));
        }
        first = false;
    }
    return QB_OK;
}

extern "C" qb_status qb_anneal_ell(qb_batch b, int32_t W, const uint32_t *tile_d, const int32_t *F0_d,
                                  const uint8_t *y0_d, int32_t nsw, int32_t B, const int32_t *thr_d, int32_t R,
                                  int32_t rw, uint64_t seed, uint32_t inst_base, uint8_t *Y_d, int64_t *e_d,
                                  void *stream)
{
    return qb_anneal_ell_x(b, W, tile_d, F0_d, y0_d, nsw, B, thr_d, R, rw, seed, inst_base, nullptr, Y_d, e_d, stream);
}
