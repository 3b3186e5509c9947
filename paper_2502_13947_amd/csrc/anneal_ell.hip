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
//
// k_anneal_ell_spec decides a whole sweep at once and repairs it;
// k_anneal_ell takes accepts one by one (a block's 64 candidates evaluated at
// once, the lowest accepting lane taken by ballot and find-first-set, lanes
// past it re-evaluated after its row was added), and serves the jobs that do
// not leave LDS for the other's tables, and rows wider than 255.
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
template <int MS>
__global__ void __launch_bounds__(1024) k_anneal_ell(const int32_t *__restrict__ jobs, int rgroups,
                                                     const int32_t *__restrict__ off, int W,
                                                     const uint32_t *__restrict__ tiles,
                                                     const int32_t *__restrict__ F0,
                                                     const uint8_t *__restrict__ y0, int nsw, int B,
                                                     const int32_t *__restrict__ thr, int R, int rw, uint32_t k0,
                                                     uint32_t k1, uint32_t inst_base, const qb_iter *__restrict__ it, uint8_t *__restrict__ Y,
                                                     int64_t *__restrict__ eout, int32_t *__restrict__ acnt)
{
    constexpr int MP = 64 * MS;
    extern __shared__ __align__(16) uint32_t dl[];
    const int q = jobs[blockIdx.x / rgroups];
    const int rg = blockIdx.x % rgroups;
    const int base = off[q], m = off[q + 1] - base;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int r = rg * rw + wid;

    uint32_t *tl = dl;                                   // [m][W]
    int32_t *F = reinterpret_cast<int32_t *>(dl + (size_t)MP * W) + wid * MP;
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(tiles + (int64_t)base * W);
        uint4 *dst = reinterpret_cast<uint4 *>(tl);
        const int n16 = m * W / 4;
        for (int t = tid; t < n16; t += blockDim.x) dst[t] = src[t];
    }
#pragma unroll
    for (int s = 0; s < MS; ++s) {
        const int pos = 64 * s + lane;
        F[pos] = pos < m ? F0[base + pos] : 0;
    }
    __syncthreads();
    if (r >= R) return;   // no barrier follows

    uint32_t ybits = 0;
    uint64_t active[MS];
#pragma unroll
    for (int s = 0; s < MS; ++s) {
        const int pos = 64 * s + lane;
        if (pos < m && y0[base + pos]) ybits |= 1u << s;
        const int na = min(max(m - 64 * s, 0), 64);
        active[s] = na == 64 ? ~0ull : ((1ull << na) - 1ull);
    }
    int64_t e = 0;
    int32_t nacc = 0;
    const uint32_t tag = (1u << 28) | (inst_base + (it ? it->inst : 0u) + (uint32_t)q);
    constexpr int G = (MS + 3) / 4;
    const int sh = 32 - B;

    for (int sw = 0; sw < nsw; ++sw) {
        uint32_t u[4 * G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint4 o = qb_philox(make_uint4(((uint32_t)g << 6) | (uint32_t)lane, (uint32_t)sw, (uint32_t)r, tag),
                                      k0, k1);
            u[4 * g + 0] = o.x;
            u[4 * g + 1] = o.y;
            u[4 * g + 2] = o.z;
            u[4 * g + 3] = o.w;
        }
        const int32_t *ts = thr + ((size_t)sw << B);
        int32_t tv[MS];
#pragma unroll
        for (int s = 0; s < MS; ++s) tv[s] = ts[u[s] >> sh];
#pragma unroll
        for (int s = 0; s < MS; ++s) {
            uint64_t pend = active[s];
            if (pend == 0) continue;
            int32_t fs = F[64 * s + lane];
            // the first 64 words of the row of lane kp, read one accept ahead:
            // kp is the next accepting lane of the current ballot, which is
            // most often the next accept, and its row read then overlaps the
            // current update instead of following it
            int kp = -1;
            uint32_t wp = 0u;
            while (true) {
                const uint32_t yb = (ybits >> s) & 1u;
                const int32_t dE = yb ? -fs : fs;
                const uint64_t acc = __ballot(dE <= tv[s]) & pend;
                if (acc == 0) break;
                const int k = __builtin_ctzll(acc);
                const int32_t dEk = __builtin_amdgcn_readlane(dE, k);
                const int32_t ykb = __builtin_amdgcn_readlane((int32_t)yb, k);
                e += dEk;
                ++nacc;
                const int32_t d2 = ykb ? -2 : 2;
                if (lane == k) ybits ^= 1u << s;
                const uint32_t *row = tl + (size_t)(64 * s + k) * W;
                // (word lane of a row is inside the LDS allocation for every
                // lane: the fields of the replicas follow the tile)
                uint32_t w0 = wp;
                if (kp != k) w0 = row[lane];
                if (lane < W && w0 != 0u) atomicAdd(&F[qb_ell_col(w0)], d2 * qb_ell_val(w0));
                for (int t0 = 64; t0 < W; t0 += 64) {
                    if (t0 + lane < W) {
                        const uint32_t wd = row[t0 + lane];
                        if (wd != 0u) atomicAdd(&F[qb_ell_col(wd)], d2 * qb_ell_val(wd));
                    }
                }
                // issued after the adds (which return nothing), so only the
                // read of the fields below waits for it
                const uint64_t rest = acc & ~((2ull << k) - 1ull);
                kp = rest ? __builtin_ctzll(rest) : -1;
                if (kp >= 0) wp = tl[(size_t)(64 * s + kp) * W + lane];
                pend &= ~((2ull << k) - 1ull);
                fs = F[64 * s + lane];
            }
        }
    }

    uint8_t *Yr = Y + (size_t)base * R + (size_t)r * m;
#pragma unroll
    for (int s = 0; s < MS; ++s) {
        const int pos = 64 * s + lane;
        if (pos < m) Yr[pos] = (uint8_t)((ybits >> s) & 1u);
    }
    if (lane == 0) eout[(size_t)q * R + r] = e;
    if (acnt && lane == 0) acnt[(size_t)q * R + r] = nacc;
}

// The same sweep, speculated: a whole sweep is decided at once and repaired
// until it agrees with the sequential one (the fixed point of evaluating
// every position against a guess of all decisions is the sequential sweep's,
// as a position's answer depends on lower positions only).  A row of a sparse
// tile reaches few positions, so almost every first guess is right: on the
// sub-QUBOs of the n = 20000 workload (1024 variables, 230 accepts a sweep)
// 2.8 rounds change anything, against a chain of 230 accepts.
//
// One wave per replica, lane L holding the positions 64 s + L.  F lives in
// LDS.  A round compares every position's field with its threshold and adds
// what the changed decisions make of the fields of *later* positions (LDS
// atomic adds); once nothing changes, the accepted rows' entries at earlier
// positions are added too.  Entries ascend by column, so a row's earlier part
// comes first; of either part the first entry is in registers, and the others
// are read from the tile in LDS by the few lanes that have any.  With F exact
// at both ends the energy of the whole run is 1/2 sum (y - y0) (F0 + F): no
// sweep sums it.  The thresholds of KT sweeps at a time are staged in LDS (KT
// = 0: read from memory), one barrier per KT sweeps.
//
// Bound by a wave's own instructions and LDS round trips (12,000 cycles a
// sweep of 1024, Philox 2200 of them; 16 replicas take as long as one).
// Measured, 128 jobs x 16 replicas x 1000 sweeps: 5.1 ms, against 30.2 ms for
// a kernel that chained the accepts one by one with the block's couplings in
// registers.
__device__ __forceinline__ int32_t sat_add(int32_t a, int32_t b) { return __builtin_elementwise_add_sat(a, b); }

template <int MS, bool TLDS>
__global__ void __launch_bounds__(512) k_anneal_ell_spec(const int32_t *__restrict__ jobs, int rgroups,
                                                         const int32_t *__restrict__ off, int W,
                                                         const uint32_t *__restrict__ tiles,
                                                         const int32_t *__restrict__ F0,
                                                         const uint8_t *__restrict__ y0, int nsw, int B,
                                                         const int32_t *__restrict__ thr, int KT, int R, int rw,
                                                         uint32_t k0, uint32_t k1, uint32_t inst_base,
                                                         const qb_iter *__restrict__ it, uint8_t *__restrict__ Y,
                                                         int64_t *__restrict__ eout, int32_t *__restrict__ acnt)
{
    constexpr int MP = 64 * MS, NPRE = 8;
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
    int32_t *ts = Fall + rw * MP;                                 // [2][KT][2^B]
    uint16_t *info = reinterpret_cast<uint16_t *>(ts + (TLDS ? (size_t)2 * KT << B : 0));   // [MP] entries: earlier, all
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(tiles + (int64_t)base * W);
        uint4 *dst = reinterpret_cast<uint4 *>(tl);
        const int n16 = m * W / 4;
        for (int t = tid; t < n16; t += nt) dst[t] = src[t];
        if constexpr (TLDS) {
            const int n = min(KT, nsw) << B;
            for (int t = tid; t < n; t += nt) ts[t] = thr[t];
        }
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
        info[a] = (uint16_t)(nu | (cnt << 8));
    }
    int32_t M[MS];                          // -y
    uint32_t yb = 0;
#pragma unroll
    for (int s = 0; s < MS; ++s) {
        const int pos = 64 * s + lane;
        if (live) F[pos] = pos < m ? F0[base + pos] : 0;
        if (pos < m && y0[base + pos]) yb |= 1u << s;
        M[s] = (yb >> s) & 1u ? -1 : 0;
    }
    const uint32_t y00 = yb;
    __syncthreads();

    // first entries: twice the coupling, and the byte offset of the field it
    // moves (none: zero into the position's own field)
    const uint32_t fo = (uint32_t)(reinterpret_cast<char *>(F) - reinterpret_cast<char *>(dl));
    int32_t dv[MS], uv[MS];
    uint32_t da[MS], ua[MS];
    uint32_t hd = 0, hd2 = 0, hu = 0, hu2 = 0;   // positions with one, and with more, later or earlier entries
#pragma unroll
    for (int s = 0; s < MS; ++s) {
        const int pos = 64 * s + lane;
        const int nu = info[pos] & 255, nd = (info[pos] >> 8) - nu;
        const uint32_t wu = nu > 0 ? tl[pos * W] : 0u, wd = nd > 0 ? tl[pos * W + nu] : 0u;
        uv[s] = 2 * qb_ell_val(wu);
        ua[s] = fo + 4u * (uint32_t)(nu > 0 ? qb_ell_col(wu) : pos);
        dv[s] = 2 * qb_ell_val(wd);
        da[s] = fo + 4u * (uint32_t)(nd > 0 ? qb_ell_col(wd) : pos);
        hu |= (uint32_t)(nu > 0) << s;
        hu2 |= (uint32_t)(nu > 1) << s;
        hd |= (uint32_t)(nd > 0) << s;
        hd2 |= (uint32_t)(nd > 1) << s;
    }
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
            const int nu = info[pos] & 255, cnt = info[pos] >> 8;
            const int32_t f = (neg >> s) & 1u ? -2 : 2;
            const uint32_t *row = tl + pos * W;
            for (int t = (later ? nu : 0) + skip; t < (later ? cnt : nu); ++t) {
                const uint32_t wd = row[t];
                atomicAdd(F + qb_ell_col(wd), f * qb_ell_val(wd));
            }
        }
    };

    int32_t nacc = 0;
    const uint32_t tag = (1u << 28) | (inst_base + (it ? it->inst : 0u) + (uint32_t)q);
    constexpr int G = (MS + 3) / 4;
    const int sh = 32 - B;
    const int chunk = TLDS ? KT : nsw;
    for (int c0 = 0; c0 < nsw; c0 += chunk) {
        const int nc = min(chunk, nsw - c0), buf = TLDS ? (c0 / chunk) & 1 : 0;
        // the next chunk's thresholds, on their way while this one is swept
        int32_t pre[NPRE];
        const int nn = TLDS ? max(min(chunk, nsw - c0 - nc), 0) << B : 0;
        if constexpr (TLDS) {
#pragma unroll
            for (int i = 0; i < NPRE; ++i)
                if (tid + i * nt < nn) pre[i] = thr[((size_t)(c0 + nc) << B) + tid + i * nt];
        }
        if (live) {
#pragma unroll 1
            for (int sw = c0; sw < c0 + nc; ++sw) {
                int32_t tp[MS];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const uint4 o = qb_philox(make_uint4(((uint32_t)g << 6) | (uint32_t)lane, (uint32_t)sw, (uint32_t)r,
                                                         tag), k0, k1);
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        if (4 * g + w < MS) {
                            const uint32_t k = qb_word(o, w) >> sh;
                            tp[4 * g + w] = TLDS ? ts[((buf * KT + sw - c0) << B) + k] : thr[((size_t)sw << B) + k];
                        }
                }
                // dE <= t on x = F ^ -y: for y = 1, -F <= t is ~F <= t - 1 (no
                // field reaches INT32_MAX, nor a position past the job INT32_MIN)
#pragma unroll
                for (int s = 0; s < MS; ++s) tp[s] = 64 * s + lane < m ? sat_add(tp[s], M[s]) : INT32_MIN;
                auto decide = [&]() {
                    uint32_t a = 0;
#pragma unroll
                    for (int s = MS - 1; s >= 0; --s) a = 2 * a + (uint32_t)((F[64 * s + lane] ^ M[s]) <= tp[s]);
                    return a;
                };
                uint32_t acc = decide();
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
                nacc += __builtin_popcount(acc);
                yb ^= acc;
#pragma unroll
                for (int s = 0; s < MS; ++s) M[s] = -(int32_t)((yb >> s) & 1u);
            }
        }
        if constexpr (TLDS) {
            if (nn > 0) {
                int32_t *dst = ts + ((size_t)((buf ^ 1) * KT) << B);
#pragma unroll
                for (int i = 0; i < NPRE; ++i)
                    if (tid + i * nt < nn) dst[tid + i * nt] = pre[i];
                for (int t = tid + NPRE * nt; t < nn; t += nt) dst[t] = thr[((size_t)(c0 + nc) << B) + t];
                __syncthreads();
            }
        }
    }
    if (!live) return;

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

// Sweeps whose thresholds the speculating kernel stages at a time: as many as
// fit (at most 4), 0 to read them from memory; -1 where the job's rows, the
// fields and the entry counts do not fit.
inline int ell_spec_stage(int ms, int W, int rw, int B, size_t *bytes)
{
    const size_t need = sizeof(uint32_t) * ((size_t)64 * ms * (W + rw)) + sizeof(uint16_t) * 64 * ms;
    for (int k = 4; k >= 0; k >>= 1) {
        *bytes = need + (B <= 12 ? ((size_t)2 * k * sizeof(int32_t)) << B : 0);
        if (k > 0 && B > 12) continue;
        if (*bytes <= LDS_MAX) return k;
        if (k == 0) break;
    }
    return -1;
}

template <int MS>
qb_status launch_ell(int njobs, int rw, int R, hipStream_t s, const int32_t *jobs, qb_batch b, int W,
                     const uint32_t *tiles, const int32_t *F0, const uint8_t *y0, int nsw, int B, const int32_t *thr,
                     uint64_t seed, uint32_t inst_base, const qb_iter *it, uint8_t *Y, int64_t *e)
{
    const size_t lds = ell_lds_bytes(MS, W, rw);
    size_t slds = 0;
    // up to 8 replicas per workgroup (256 registers a lane), more in further workgroups
    const int srw = rw < 8 ? rw : 8;
    const int kt = W <= 255 ? ell_spec_stage(MS, W, srw, B, &slds) : -1;
    if (kt >= 0) {
        const int rgroups = (R + srw - 1) / srw;
        const auto kern = kt > 0 ? k_anneal_ell_spec<MS, true> : k_anneal_ell_spec<MS, false>;
        QB_TRY_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_MAX));
        kern<<<njobs * rgroups, 64 * srw, slds, s>>>(jobs, rgroups, b->off_d, W, tiles, F0, y0, nsw, B, thr, kt, R, srw,
                                                     (uint32_t)seed, (uint32_t)(seed >> 32), inst_base, it, Y, e,
                                                     b->acnt_d);
        QB_LAUNCH_CHECK();
        return QB_OK;
    }
    // set on every launch (no cached flag shared between devices or threads)
    QB_TRY_HIP(hipFuncSetAttribute((const void *)k_anneal_ell<MS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)LDS_MAX));
    const int rgroups = (R + rw - 1) / rw;
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
