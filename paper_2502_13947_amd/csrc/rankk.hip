// Rank-k local-field update H[p] += Q dX[p] (the Tabu section's O(n)
// move-value update generalised to every variable a stage changed).
//
// VALU variant (any Q, best for few solutions): a workgroup has 1024 columns
// of one solution and a range of rows; the changed variables of the range are
// compacted into an LDS list and every thread adds +-Q[j][i] for its four
// consecutive columns (Q is symmetric, so column j of Q is row j).
#include <math.h>

#include <algorithm>

#include "qb_internal.h"

namespace {

// What bounds it: the chain of row loads, so the rows are split over
// blockIdx.z until the card is full (partial sums added with integer atomics:
// exact, any order) and eight of a thread's loads are in flight at once.
// RK_ROWS of the range are compacted at a time
// (n = 2500, 4 solutions: 68 us unsplit with one load in flight, 5.3 us so).
constexpr int RK_ROWS = 256;

template <typename QT>
__global__ void __launch_bounds__(256) k_rankk_valu(const QT *__restrict__ Q, int n, const int8_t *__restrict__ dX,
                                                    int32_t *__restrict__ H, int rows)
{
    __shared__ int32_t list[RK_ROWS + 7];            // padded to a multiple of 8 with 0 = no row
    __shared__ int wcnt[4];
    const int p = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = blockIdx.x * 1024 + 4 * tid;
    const int8_t *d = dX + (int64_t)p * n;
    const int jb = blockIdx.z * rows, je = min(jb + rows, n);
    int32_t acc[4] = {0, 0, 0, 0};
    for (int j0 = jb; j0 < je; j0 += RK_ROWS) {
        const int j = j0 + tid;
        const int v = j < je ? d[j] : 0;
        const uint64_t mask = __ballot(v != 0);
        if (lane == 0) wcnt[wave] = __popcll(mask);
        __syncthreads();
        int base = 0, cnt = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            base += w < wave ? wcnt[w] : 0;
            cnt += wcnt[w];
        }
        if (v) list[base + __popcll(mask & ((1ull << lane) - 1))] = v > 0 ? (j + 1) : -(j + 1);
        if (tid < 7) list[cnt + tid] = 0;
        __syncthreads();
        if (i + 4 <= n) {
            for (int u = 0; u < cnt; u += 8) {
                QT q[8][4];                          // one load each, at any alignment
                int32_t sg[8];
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const int32_t e = __builtin_amdgcn_readfirstlane(list[u + v]);
                    sg[v] = e > 0 ? 1 : e < 0 ? -1 : 0;
                    __builtin_memcpy(q[v], Q + (int64_t)(e > 0 ? e - 1 : e < 0 ? -e - 1 : 0) * n + i, sizeof q[v]);
                }
#pragma unroll
                for (int v = 0; v < 8; ++v)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] += sg[v] * (int32_t)q[v][c];
            }
        } else if (i < n) {                          // the last, partial group of columns
            for (int u = 0; u < cnt; ++u) {
                const int32_t e = list[u];
                const int32_t sg = e < 0 ? -1 : 1;
                const QT *row = Q + (int64_t)(e < 0 ? -e - 1 : e - 1) * n;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (i + c < n) acc[c] += sg * (int32_t)row[i + c];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (acc[c]) {                                // never past n: those sums stay 0
            int32_t *h = &H[(int64_t)p * n + i + c];
            if (gridDim.z == 1) *h += acc[c];
            else atomicAdd(h, acc[c]);
        }
}

// ------------------------------------------------------------------ MFMA variant
// H (z x n) += dX (z x n, int8) . Q (n x n, int8): a real dense contraction.
// Q is symmetric, so the B operand's column i is row i of the padded copy Qp
// (K-contiguous, like the A operand's rows of dX).  v_mfma_i32_16x16x64_i8
// with int32 accumulation is exact (|sum| <= n * 127 * 1).
//
// What bounds it: reading Q once (n*n bytes) and feeding the matrix cores.  A
// workgroup has 64*WM solutions (all of up to 256, so that Q is read once) x
// 128 columns, a wave 64 x 64 of them.  Steps of 128 rows go from memory to
// registers two steps ahead and through two LDS buffers, so that every row is
// read once per workgroup in whole 128-byte lines; rows of 144 bytes in LDS
// give the 16-byte operand reads of 16 lanes distinct banks.  K is split over
// blockIdx.z and the partial sums are added with integer atomics (exact and
// order independent).  A call of n = 7000, 256 solutions: 76 us with 64
// solutions per workgroup and operands straight from memory, 46 us so.
typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int RM_K = 128, RM_N = 128, RM_LD = RM_K + 16;

// 16 bytes of a row of dX at kk, zero from n on, without a branch on a lane:
// the row's last 16 bytes shifted into place where kk + 16 passes its end
// (rows start at any byte: one load at any alignment)
__device__ __forceinline__ v4i load_end16(const int8_t *__restrict__ row, int kk, int n)
{
    uint64_t w[2] = {0, 0};
    if (n >= 16) {
        const int at = min(kk, n - 16), sh = 8 * min(kk - at, 16);
        __builtin_memcpy(w, row + at, 16);
        const uint64_t lo = sh < 64 ? w[0] >> sh : 0, up = sh == 0 || sh >= 128 ? 0 : sh < 64 ? w[1] << (64 - sh)
                                                                                          : w[1] >> (sh - 64);
        w[0] = lo | up;
        w[1] = sh < 64 ? w[1] >> sh : 0;
    } else {
#pragma unroll
        for (int b = 0; b < 16; ++b) {
            const uint64_t v = (uint8_t)row[min(kk + b, n - 1)];
            w[b >> 3] |= kk + b < n ? v << (8 * (b & 7)) : 0;
        }
    }
    v4i v;
    __builtin_memcpy(&v, w, 16);
    return v;
}

template <int WM>
__global__ void __launch_bounds__(128 * WM) k_rankk_mfma(const int8_t *__restrict__ dX, int n, int z,
                                                         const int8_t *__restrict__ Qp, int ldp,
                                                         int32_t *__restrict__ H, int kchunk)
{
    constexpr int TB = 128 * WM, RPT = TB / 8;       // rows loaded by one round of the workgroup
    constexpr int NA = 64 * WM / RPT, NB = RM_N / RPT;
    __shared__ __align__(16) int8_t la[2][64 * WM][RM_LD];
    __shared__ __align__(16) int8_t lb[2][RM_N][RM_LD];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int m0 = blockIdx.y * (64 * WM), n0 = blockIdx.x * RM_N;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    const int kpad = (n + 63) & ~63;                 // Qp is zero from n to here
    const int kbeg = blockIdx.z * kchunk;
    const int nstep = (min(kchunk, kpad - kbeg) + RM_K - 1) / RM_K;
    const int r16 = lane & 15, g = lane >> 4;
    const int lrow = tid >> 3, lcol = (tid & 7) * 16;
    // rows past the last solution or variable are read as the first one: their
    // sums are not stored
    const int8_t *ap[NA], *bp[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int p = m0 + lrow + i * RPT;
        ap[i] = dX + (int64_t)(p < z ? p : 0) * n;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int c = n0 + lrow + i * RPT;
        bp[i] = Qp + (int64_t)(c < n ? c : 0) * ldp;
    }
    struct Stage { v4i a[NA], b[NB]; };
    auto fetch = [&](Stage &st, int step) {
        const int kk = kbeg + step * RM_K + lcol;
        if (kbeg + (step + 1) * RM_K <= n) {         // no condition on a lane, so no wait between the loads
#pragma unroll
            for (int i = 0; i < NA; ++i) __builtin_memcpy(&st.a[i], ap[i] + kk, 16);
#pragma unroll
            for (int i = 0; i < NB; ++i) st.b[i] = *reinterpret_cast<const v4i *>(bp[i] + kk);
        } else if (step < nstep) {                   // the step that holds the rows' ends
#pragma unroll
            for (int i = 0; i < NA; ++i) st.a[i] = load_end16(ap[i], kk, n);
#pragma unroll
            for (int i = 0; i < NB; ++i)
                st.b[i] = *reinterpret_cast<const v4i *>(bp[i] + min(kk, kpad - 16));   // past n: times 0
        }
    };
    auto stash = [&](const Stage &st, int buf) {
#pragma unroll
        for (int i = 0; i < NA; ++i) *reinterpret_cast<v4i *>(&la[buf][lrow + i * RPT][lcol]) = st.a[i];
#pragma unroll
        for (int i = 0; i < NB; ++i) *reinterpret_cast<v4i *>(&lb[buf][lrow + i * RPT][lcol]) = st.b[i];
    };
    v4i acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = v4i{0, 0, 0, 0};
    auto multiply = [&](int buf) {
#pragma unroll
        for (int k = 0; k < RM_K; k += 64) {
            v4i a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = *reinterpret_cast<const v4i *>(&la[buf][wm + 16 * i + r16][k + 16 * g]);
#pragma unroll
            for (int i = 0; i < 4; ++i) b[i] = *reinterpret_cast<const v4i *>(&lb[buf][wn + 16 * i + r16][k + 16 * g]);
#pragma unroll
            for (int mi = 0; mi < 4; ++mi)
#pragma unroll
                for (int ni = 0; ni < 4; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[mi], b[ni], acc[mi][ni], 0, 0, 0);
        }
    };
    // step s is multiplied from buffer s & 1 while step s + 1 is in registers
    // or on its way and step s + 2 is asked for
    Stage s0, s1;
    fetch(s0, 0);
    fetch(s1, 1);
    stash(s0, 0);
    for (int step = 0; step < nstep; step += 2) {
        fetch(s0, step + 2);
        qb_lds_barrier();
        multiply(0);
        stash(s1, 1);
        fetch(s1, step + 3);
        qb_lds_barrier();
        if (step + 1 < nstep) multiply(1);
        stash(s0, 0);
    }
    // 16x16 result layout: lane holds rows 4g..4g+3 of column r16
#pragma unroll
    for (int mi = 0; mi < 4; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int p = m0 + wm + mi * 16 + 4 * g + r;
                const int i = n0 + wn + ni * 16 + r16;
                const int32_t v = acc[mi][ni][r];
                if (p < z && i < n && v != 0) atomicAdd(&H[(int64_t)p * n + i], v);
            }
}

template <int WM>
qb_status rankk_mfma_go(qb_problem P, int z, const int8_t *dX, int32_t *H, int split, int ncu, hipStream_t s)
{
    const int n = P->n;
    const int gx = (n + RM_N - 1) / RM_N, gy = (z + 64 * WM - 1) / (64 * WM);
    const int nk = (n + RM_K - 1) / RM_K;
    // 304 registers a lane (WM = 4: 256) leave room for one workgroup on a
    // compute unit, of two waves (WM = 1) for two.  A split more where a third
    // of the units have none: solutions that did not change add nothing (n =
    // 7000, 256 solutions: 34 and 27 us with 3 and 4 splits for none changed,
    // 36 and 32 for a third, 48 and 49 for all).
    const int wgs = gx * gy, fit = ncu * (WM == 1 ? 2 : 1);
    if (3 * wgs * split <= 2 * ncu && wgs * (split + 1) <= ncu) ++split;
    // the fewest whose workgroups take less than a tenth more steps one after
    // another than the best number's (n = 12,000, 65 solutions: 65, 60 and 62
    // us with 2, 5 and 8)
    auto chain = [&](int k) { return (wgs * k + fit - 1) / fit * ((nk + k - 1) / k); };
    int least = chain(1), k = 1;
    for (int t = 2; t <= std::min(split, nk); ++t) least = std::min(least, chain(t));
    while (10 * chain(k) >= 11 * least) ++k;
    const int steps = (nk + k - 1) / k;
    k_rankk_mfma<WM><<<dim3(gx, gy, (nk + steps - 1) / steps), 128 * WM, 0, s>>>(
        dX, n, z, (const int8_t *)P->Qp, P->ldp, H, RM_K * steps);
    QB_LAUNCH_CHECK();
    return QB_OK;
}

// Sparse product over the row-major ELL: H[p][i] (+)= Q_ii V[p][i] +
// sum_t val_t V[p][col_t].  One thread per (i, p); a row's words are read as
// 16-byte vectors (the width is a multiple of 4, and the zero words past a
// row's last entry add 0).
template <typename VT, bool ACC>
__global__ void __launch_bounds__(256) k_ell_spmm(const uint32_t *__restrict__ ell, const int32_t *__restrict__ ecnt,
                                                  const int32_t *__restrict__ diag, int n, int W,
                                                  const VT *__restrict__ V, int32_t *__restrict__ H)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int p = blockIdx.y;
    if (i >= n) return;
    const VT *v = V + (int64_t)p * n;
    int32_t acc = diag[i] * (int32_t)v[i];
    const uint4 *row = reinterpret_cast<const uint4 *>(ell + (int64_t)i * W);
    const int c4 = (ecnt[i] + 3) >> 2;
    for (int t = 0; t < c4; ++t) {
        const uint4 w = row[t];
        acc += qb_ell_val(w.x) * (int32_t)v[qb_ell_col(w.x)];
        acc += qb_ell_val(w.y) * (int32_t)v[qb_ell_col(w.y)];
        acc += qb_ell_val(w.z) * (int32_t)v[qb_ell_col(w.z)];
        acc += qb_ell_val(w.w) * (int32_t)v[qb_ell_col(w.w)];
    }
    int32_t *h = H + (int64_t)p * n + i;
    *h = ACC ? *h + acc : acc;
}

}  // namespace

qb_status qb_field_ell_launch(qb_problem P, int z, const uint8_t *X, int32_t *H, hipStream_t s)
{
    dim3 grid((P->n + 255) / 256, z);
    k_ell_spmm<uint8_t, false><<<grid, 256, 0, s>>>(P->ell, P->ecnt, P->diag, P->n, P->ellw, X, H);
    QB_LAUNCH_CHECK();
    return QB_OK;
}

qb_status qb_rankk_mfma_launch(qb_problem P, int z, const int8_t *dX, int32_t *H, hipStream_t s)
{
    int ncu = 0;
    QB_TRY_HIP(qb_cu_count(&ncu));
    // Every split spares a workgroup n / 128 / split steps of 2 us and costs z n
    // atomic additions, 7 us a million: least at 48 / sqrt(z), whatever n is
    // (n = 2500, 256 solutions: 17, 16, 19 and 20 us with 2, 3, 4 and 6; n =
    // 7000, 64: 31, 27, 26 and 26 with 3, 4, 6 and 8; n = 1000, 2048: 17, 22 and
    // 37 with 1, 2 and 4).
    const int split = std::max((int)lrint(48.0 / sqrt((double)z)), 1);
    // As many solutions a workgroup as leave at least five workgroups for
    // eight compute units (n = 5000, 256 solutions: 31 us with 128, 34 with 256
    // in a workgroup; n = 7000: 49 and 48; n = 2500: 16 with 64, 17 with 128).
    const int64_t gx = (P->n + RM_N - 1) / RM_N;
    int wm = z <= 64 ? 1 : z <= 128 ? 2 : 4;
    while (wm > 1 && 8 * gx * ((z + 64 * wm - 1) / (64 * wm)) * split < 5 * ncu) wm >>= 1;
    return wm == 1 ? rankk_mfma_go<1>(P, z, dX, H, split, ncu, s)
           : wm == 2 ? rankk_mfma_go<2>(P, z, dX, H, split, ncu, s) : rankk_mfma_go<4>(P, z, dX, H, split, ncu, s);
}

extern "C" qb_status qb_rankk(qb_problem P, int32_t z, const int8_t *dX_d, int32_t *H_d, int32_t variant,
                             void *stream)
{
    if (!P || z < 1 || z > 65535 || !dX_d || !H_d || variant < 0 || variant > 3) return QB_E_ARG;
    hipStream_t s = qb_stream(stream);
    if (P->sparse) {
        if (variant != 0 && variant != 3) return QB_E_UNSUPPORTED;
        dim3 g((P->n + 255) / 256, z);
        k_ell_spmm<int8_t, true><<<g, 256, 0, s>>>(P->ell, P->ecnt, P->diag, P->n, P->ellw, dX_d, H_d);
        QB_LAUNCH_CHECK();
        return QB_OK;
    }
    if (variant == 3 || (variant == 2 && !P->int8_ok)) return QB_E_UNSUPPORTED;
    if (variant == 0) variant = (P->int8_ok && P->Qp && z >= 32) ? 2 : 1;
    if (variant == 2) {
        if (!P->Qp) return QB_E_UNSUPPORTED;
        return qb_rankk_mfma_launch(P, z, dX_d, H_d, s);
    }
    const int gx = (P->n + 1023) / 1024;
    // rows per workgroup: a multiple of 64, so that about 1024 workgroups share the work
    const int64_t want = 1024 / ((int64_t)gx * z) > 1 ? 1024 / ((int64_t)gx * z) : 1;
    const int rows = 64 * (int)((P->n + 64 * want - 1) / (64 * want));
    dim3 grid(gx, z, (P->n + rows - 1) / rows);
    if (P->int8_ok)
        k_rankk_valu<int8_t><<<grid, 256, 0, s>>>(P->Q8, P->n, dX_d, H_d, rows);
    else
        k_rankk_valu<int16_t><<<grid, 256, 0, s>>>(P->Q, P->n, dX_d, H_d, rows);
    QB_LAUNCH_CHECK();
    return QB_OK;
}
