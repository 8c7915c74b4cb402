// Partitioned factorization of the shifted band (gfx950).
//
// The Cayley transform of Sec. 2 needs one factorization of C = A - sigma B per shift;
// a whole-matrix band LU is a chain of n/16 dependent panel steps.  Here C is split as
// C = D + E, D block diagonal (diagonal blocks D_j of bs columns, the last one shorter)
// and E the couplings between neighbouring blocks, in the divide-and-conquer form of the
// SPIKE algorithm (Polizzi and Sameh):
//   * every D_j is factored with partial pivoting inside the block, all blocks in the
//     same launches (the band LU in its block-diagonal mode), so a factor takes bs/16
//     panel steps instead of n/16;
//   * the spikes V = D^{-1} E_up, W = D^{-1} E_low: with boundary q_p = (p+1) bs, column
//     k of V holds, in the rows of block p, D_p^{-1} times the coupling of block p to
//     x[q_p + k] (k < ku); column k of W holds, in the rows of block p+1, D_{p+1}^{-1}
//     times the coupling of block p+1 to x[q_p - kl + k] (k < kl);
//   * the reduced system: with t_p = x[q_p .. q_p + ku) and b_p = x[q_p - kl .. q_p), the
//     rows of x = g - V t - W b at the tips give, per boundary p,
//         b_p + V(b rows) t_p + W(b rows) b_{p-1} = g(b rows)
//         t_p + W(t rows) b_p + V(t rows) t_{p+1} = g(t rows),
//     a band system R of order nr = (nbk - 1)(kl + ku) with lower bandwidth 2 kl + ku - 1
//     and upper kl + 2 ku - 1, nr <= 4096.  Its inverse is put together from the
//     boundaries' own (kl + ku) x (kl + ku) blocks by merging neighbours pairwise (below);
//   * a solve C y = u is g = D^{-1} u (the partitioned sweeps of D's factor), z = R^{-1}
//     tips(g), and y_i = g_i - sum_k V[i,k] t[k] - sum_k W[i,k] b[k] with the tips of the
//     boundaries of row i's block.
// Pivoting never crosses a block boundary, so the caller checks the backward error of a
// solve and factors the whole matrix instead when it is not small.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "common.hpp"
#include "kernels.hpp"

namespace simm {

namespace {
constexpr int kLdsMaxW = 64;      // widest kl + ku inverted inside one workgroup
constexpr int kShortMaxW = 128;   // widest kl + ku of blocks shorter than 1,024 rows
constexpr int64_t kReducedFill = 2048;   // reduced order filled with blocks without weighing their cost
constexpr double kApplications = 80.0;   // solves a factor is made for (the steps of a Krylov space)
constexpr int kMergeMaxW = 512;   // widest kl + ku of a partitioned factor (k_gj_step's rows)
}

int64_t part_block_len(int64_t n, int kl, int ku) {
    const int w = kl + ku;
    if (kl < 1 || ku < 1) return 0;
    if (w > kMergeMaxW) return 0;
    int64_t bs = -1;
    if (const char* e = getenv("SIMM_LU_PART")) bs = atoll(e);   // 0: never; > 0: this block length
    if (bs == 0) return 0;
    // each block holds both tips of its boundaries, and a workgroup of the sweeps'
    // corrections (256 rows) spans at most two blocks
    const int64_t bmin = std::max<int64_t>(256, (2 * (int64_t)w + 15) / 16 * 16);
    if (bs > 0) {
        bs = std::max<int64_t>((bs + 15) / 16 * 16, bmin);
    } else {
        // As many blocks as keep the reduced order within 2,048.  Up to w = kShortMaxW blocks go
        // down to max(256, 4 w) rows: a block is then a chunk or few of the sweeps and the LU
        // has bs / 16 panel steps (n = 14,167, k = 16: 50 blocks of 288 rows, an application
        // 114 us and a factor 4.3 ms against 199 us and 5.3 ms with 13 blocks of 1,104 in
        // several chunks and chains, both with the chunk sweeps of then; 76 us now).  Wider couplings take w / 16 panel steps per level of the
        // reduced inverse: blocks of at least max(1024, 4 w) rows.
        const int64_t rows = std::max<int64_t>(w <= kShortMaxW ? 256 : 1024, 4 * (int64_t)w);
        int64_t nb = std::min<int64_t>(1 + kReducedFill / w, n / rows);
        if (nb < 2) return 0;
        // More of them where a factor with kApplications solves is estimated at least 5 %
        // faster: half the panel steps and shorter chains of chunks against a larger inverse.
        auto len = [&](int64_t q) { return std::max<int64_t>(((n + q - 1) / q + 15) / 16 * 16, bmin); };
        auto cost = [&](int64_t q) {
            const double nr = (double)(q - 1) * w, levels = std::ceil(std::log2((double)q));
            double sweeps = 0.0;
            if (spike_block_chunks(len(q), q, kl, w, &sweeps) == 0) return 1e300;
            return (double)(len(q) / 16) * (27.0 + 0.012 * w) + levels * w * 2.0 +
                   nr * nr * w * 8.0 / 2.0e7 + kApplications * (sweeps + nr * nr * 16.0 / 5.0e6);   // us
        };
        const int64_t nb_max = std::min<int64_t>(1 + kPartMaxReduced / w, n / rows);
        double best = 0.95 * cost(nb);
        for (int64_t q = nb + 1; q <= nb_max; ++q) {
            const double c = cost(q);
            if (c < best) {
                best = c;
                nb = q;
            }
        }
        bs = len(nb);
    }
    // the last block holds at least kl + ku rows
    for (int it = 0; it < 4096 && bs < n; ++it) {
        const int64_t nbk = (n + bs - 1) / bs;
        if (n - (nbk - 1) * bs >= w) break;
        bs += 16;
    }
    if (bs >= n) return 0;
    const int64_t nbk = (n + bs - 1) / bs;
    if ((nbk - 1) * (int64_t)w > kPartMaxReduced) return 0;
    return bs;
}

size_t part_cpl_elems(int64_t n, int kl, int ku, int64_t bs) {
    const int64_t nbk = (n + bs - 1) / bs;
    return (size_t)(nbk - 1) * ((size_t)ku * ku + (size_t)kl * kl);
}

namespace {

// One workgroup per boundary q = (p+1) bs: the coupling entries C(q - ku + i, q + k)
// (k <= i) and C(q + i, q - kl + k) (i <= k) out of the band, zeroed there.
template <typename CT>
__global__ __launch_bounds__(256) void k_part_cut(int64_t n, int kl, int ku, CT* __restrict__ AB, int64_t bs,
                                                  cplx* __restrict__ cpl) {
    const int p = blockIdx.x;
    const int64_t q = (int64_t)(p + 1) * bs;
    const int kv = kl + ku, ldab = 2 * kl + ku + 1;
    cplx* cu = cpl + (size_t)p * ((size_t)ku * ku + (size_t)kl * kl);
    cplx* cl = cu + (size_t)ku * ku;
    for (int e = threadIdx.x; e < ku * ku + kl * kl; e += blockDim.x) {
        int64_t row, col;
        bool valid;
        cplx* dst;
        if (e < ku * ku) {
            const int i = e % ku, k = e / ku;
            row = q - ku + i;
            col = q + k;
            valid = k <= i && col < n;
            dst = cu + e;
        } else {
            const int e2 = e - ku * ku;
            const int i = e2 % kl, k = e2 / kl;
            row = q + i;
            col = q - kl + k;
            valid = i <= k && row < n;
            dst = cl + e2;
        }
        cplx v = mk(0.0, 0.0);
        if (valid) {
            CT* at = AB + (int64_t)(kv + row - col) + col * ldab;
            v = widen(*at);
            *at = narrow<CT>(mk(0.0, 0.0));
        }
        *dst = v;
    }
}

// Right-hand sides of the spikes, one column per blockIdx.y: the upper couplings (columns
// 0 .. ku-1, rows q_p - ku .. q_p - 1 of block p), then the lower ones (kl columns, rows q_p ..
// q_p + kl - 1 of block p+1), zero elsewhere; all n16 rows written.
__global__ __launch_bounds__(256) void k_part_rhs(int64_t n, int64_t n16, int kl, int ku, int64_t bs, int64_t nbk,
                                                  const cplx* __restrict__ cpl, cplx* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n16) return;
    const int which = (int)blockIdx.y < ku ? 0 : 1, k = which == 0 ? blockIdx.y : blockIdx.y - ku;
    cplx v = mk(0.0, 0.0);
    if (i < n) {
        const int64_t j = (unsigned)i / (unsigned)bs;
        const size_t per = (size_t)ku * ku + (size_t)kl * kl;
        if (which == 0) {
            const int64_t q = (j + 1) * bs;
            if (j <= nbk - 2 && i >= q - ku) v = cpl[(size_t)j * per + (size_t)(i - (q - ku)) + (size_t)k * ku];
        } else {
            const int64_t q = j * bs;
            if (j >= 1 && i < q + kl) v = cpl[(size_t)(j - 1) * per + (size_t)ku * ku + (size_t)(i - q) + (size_t)k * kl];
        }
    }
    out[(int64_t)blockIdx.y * n16 + i] = v;
}

__global__ void k_fill_i32(int* p, int v) {
    if (threadIdx.x == 0) *p = v;
}

// ---------------------------------------------------------------------------
// R^{-1} by pairwise merging.  For a range of boundaries let M be the
// inverse of R restricted to them.  Two neighbouring ranges with inverses M1, M2 are
// coupled by E (the t rows of the last boundary on the left to the first t on the right)
// and F (the b rows of the first boundary on the right to the last b on the left), so with
// alpha = x2[t], beta = x1[b]
//     x1 = M1 y1 - (M1[:, t] E) alpha,   x2 = M2 y2 - (M2[:, b] F) beta,
//     S [beta; alpha] = [M1[b, :] y1; M2[t, :] y2],   S = I + [0, (M1[:,t] E)[b]; (M2[:,b] F)[t], 0],
//     M = diag(M1, M2) - P (S^{-1} Q),  P = [0, M1[:, t] E; M2[:, b] F, 0], Q = [M1[b, :], 0; 0, M2[t, :]].
// All ranges of a level are merged in the same launches; the products P Z run on the FP64
// matrix cores.  A band LU of R is a chain of nr / 16 panel steps of 29 us and its
// column-by-column inverse a chain of 2 nr steps: at nr = 2,048, kl + ku = 128 the two
// took 9.9 ms, merging takes 1.9 ms (nr = 2,048, kl + ku = 64: 9.6 and 1.1 ms).
// ---------------------------------------------------------------------------

// Inverse of the w x w matrix held by the workgroup, thread (r = tid % 64, g = tid / 64)
// with entries (r, 16 g + c), the identity past w: Gauss-Jordan with partial pivoting,
// rows not moved; returns with row r of the working array holding row vk of the inverse and
// column j belonging to column plist[j] (LDS).  False if a pivot column is zero.
__device__ bool gauss_jordan(cplx (&a)[16], int w, cplx (*colb)[kLdsMaxW], cplx* rowb, int* plist, int& vk) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int r = tid % kLdsMaxW, g = tid / kLdsMaxW;
    unsigned long long used = 0;
    vk = 0;
    bool ok = true;
    for (int g0 = 0; g0 < kLdsMaxW / 16; ++g0) {
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            // (no early exit: the loop has to unroll, or `a` would be indexed by a variable)
            const int k = 16 * g0 + kk;
            if (k < w && ok) {
                cplx* cb = colb[k & 1];
                if (g == g0) cb[r] = a[kk];
                lds_barrier();
                // the largest |re| + |im| of the unused rows, first row on ties; every
                // wavefront forms it for itself
                const double v = ((used >> lane) & 1) ? -1.0 : cabs1(cb[lane]);
                const double best = wave_max(v);
                const unsigned long long bal = __ballot(v == best);
                const int p = bal ? __ffsll((long long)bal) - 1 : -1;
                ok = best > 0.0 && p >= 0;
                if (ok) {
                    const cplx inv = crecip(cb[p]);
                    if (r == p) {
#pragma unroll
                        for (int c = 0; c < 16; ++c) a[c] = a[c] * inv;
                        if (g == g0) a[kk] = inv;
#pragma unroll
                        for (int c = 0; c < 16; ++c) rowb[16 * g + c] = a[c];
                        vk = k;
                        if (g == 0) plist[k] = p;
                    }
                    lds_barrier();
                    if (r != p) {
                        const cplx f = cb[r];
                        if (g == g0) a[kk] = mk(0.0, 0.0);
#pragma unroll
                        for (int c = 0; c < 16; ++c) a[c] = fms(a[c], f, rowb[16 * g + c]);
                    }
                    used |= 1ull << p;
                }
            }
        }
    }
    lds_barrier();
    return ok;
}

// The same inverse for wider matrices, in place in global memory: wp x wp by columns (wp a
// multiple of 16, the identity past w), `batch` of them in every launch (blockIdx.y).
// Launch b has the columns of panel b (16 of them, factored by launch b - 1) eliminate all
// other columns, four per workgroup; workgroup 0 takes panel b + 1 and then factors it:
// Gauss-Jordan steps with partial pivoting over the unused rows, one row per thread.  vk[r] is
// the step that row r was the pivot of (-1: none yet), plist[k] the pivot row of step k; at
// the end row r holds row vk[r] of the inverse, column j its column plist[j].  Bound by the
// 16 dependent column steps of a panel: 24 us a launch at w = 128, 34 us at w = 400, 0.2 and
// 0.85 ms a level; inside one workgroup of 1,024 threads w = 128 took 0.49 ms.  (The band LU
// of the reduced system with its column-by-column inverse did not reach w = 400: the
// 200 x 200 grid's factor was one chain of 2,500 panel steps, 74 ms, and is now 11 blocks of
// 228 steps, 8 ms, with 9.4 ms of spikes and 7 ms of reduced inverse.)
template <int T, int NC>
__device__ __forceinline__ void gj_update(cplx (&a)[NC], const cplx* M, int wp, int b, int j0, int rc,
                                          const int* vk, const int* plist, cplx* rows) {
#pragma unroll
    for (int c = 0; c < NC; ++c) a[c] = M[rc + (int64_t)(j0 + c) * wp];
    if (b < 0) return;
    cplx p[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) p[q] = M[rc + (int64_t)(16 * b + q) * wp];
    const int v = vk[rc];
    for (int e = threadIdx.x; e < 16 * NC; e += T)
        rows[e] = M[plist[16 * b + e % 16] + (int64_t)(j0 + e / 16) * wp];
    __syncthreads();
    const bool pivot = v >= 16 * b && v < 16 * b + 16;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        cplx acc = pivot ? mk(0.0, 0.0) : a[c];
#pragma unroll
        for (int q = 0; q < 16; ++q) acc = fma_c(acc, p[q], rows[16 * c + q]);
        a[c] = acc;
    }
}

template <int T>
__global__ __launch_bounds__(T) void k_gj_step(int wp, int b, cplx* __restrict__ Ms, int* __restrict__ vks,
                                               int* __restrict__ plists, int* __restrict__ info) {
    __shared__ cplx rows[256], colb[2][T], rowb[16];
    cplx* M = Ms + (int64_t)blockIdx.y * wp * wp;
    int* vk = vks + (int64_t)blockIdx.y * wp;
    int* plist = plists + (int64_t)blockIdx.y * wp;
    const int r = threadIdx.x, lane = r & 63, rc = min(r, wp - 1);
    const bool mine = r < wp;
    if (blockIdx.x > 0) {
        const int j0 = 4 * ((int)blockIdx.x - 1);
        if (b < 0 || (j0 >> 4) == b || (j0 >> 4) == b + 1) return;
        cplx a[4];
        gj_update<T, 4>(a, M, wp, b, j0, rc, vk, plist, rows);
        if (mine) {
#pragma unroll
            for (int c = 0; c < 4; ++c) M[r + (int64_t)(j0 + c) * wp] = a[c];
        }
        return;
    }
    const int k0 = 16 * (b + 1);
    if (k0 >= wp) return;
    cplx a[16];
    gj_update<T, 16>(a, M, wp, b, k0, rc, vk, plist, rows);
    unsigned used = 0;                          // bit u: row 64 u + lane is past the matrix or was a pivot
#pragma unroll
    for (int u = 0; u < T / 64; ++u) {
        const int row = 64 * u + lane;
        if (row >= wp || vk[min(row, wp - 1)] >= 0) used |= 1u << u;
    }
    bool ok = true;
    int mystep = -1;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
        cplx* cb = colb[kk & 1];
        cb[r] = a[kk];
        lds_barrier();
        // the largest |re| + |im| of the unused rows, first row on ties; every wavefront
        // forms it for itself
        double v[T / 64], best = -1.0;
#pragma unroll
        for (int u = 0; u < T / 64; ++u) {
            const double m = cabs1(cb[lane + 64 * u]);
            v[u] = ((used >> u) & 1) ? -1.0 : m;
            best = fmax(best, v[u]);
        }
        best = wave_max(best);
        int p = -1;
#pragma unroll
        for (int u = T / 64 - 1; u >= 0; --u) {
            const unsigned long long bal = __ballot(v[u] == best);
            if (bal) p = 64 * u + __ffsll((long long)bal) - 1;
        }
        if (!(best > 0.0) || p < 0) {           // zero (or NaN) column: the caller drops the result
            ok = false;
            p = 0;
        }
        const cplx inv = crecip(cb[p]);
        if (r == p) {
#pragma unroll
            for (int c = 0; c < 16; ++c) a[c] = a[c] * inv;
            a[kk] = inv;
#pragma unroll
            for (int c = 0; c < 16; ++c) rowb[c] = a[c];
            mystep = k0 + kk;
            plist[k0 + kk] = p;
        }
        lds_barrier();
        if (r != p) {
            const cplx f = cb[r];
            a[kk] = mk(0.0, 0.0);
#pragma unroll
            for (int c = 0; c < 16; ++c) a[c] = fms(a[c], f, rowb[c]);
        }
        if ((p & 63) == lane) used |= 1u << (p >> 6);
    }
    if (!ok && r == 0) *info = 1;
    if (mine) {
#pragma unroll
        for (int c = 0; c < 16; ++c) M[r + (int64_t)(k0 + c) * wp] = a[c];
        if (mystep >= 0) vk[r] = mystep;
    }
}

// Matrix q to be inverted by the steps: I plus, in the columns j >= kl of the rows r < kl,
// ub[q sub + r rub + (j - kl) cub], and in the columns j < kl of the rows kl <= r < w,
// lb[q slb + (r - kl) rlb + j clb]; vk set to none.
__global__ __launch_bounds__(256) void k_gj_fill(int w, int kl, int wp, const cplx* __restrict__ ub, int64_t sub,
                                                 int64_t rub, int64_t cub, const cplx* __restrict__ lb, int64_t slb,
                                                 int64_t rlb, int64_t clb, cplx* __restrict__ Ms,
                                                 int* __restrict__ vks) {
    const int64_t q = blockIdx.y;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= wp * wp) return;
    const int r = e % wp, j = e / wp;
    cplx v = mk(r == j ? 1.0 : 0.0, 0.0);
    if (r < kl && j >= kl && j < w) v = ub[q * sub + r * rub + (j - kl) * cub];
    if (r >= kl && r < w && j < kl) v = lb[q * slb + (r - kl) * rlb + j * clb];
    Ms[q * wp * wp + e] = v;
    if (e < wp) vks[q * wp + e] = -1;
}

// The inverses in their place: entry (vk[r], plist[j]) at out[q sout + vk[r] ldo + plist[j]].
__global__ __launch_bounds__(256) void k_gj_out(int w, int wp, const cplx* __restrict__ Ms,
                                                const int* __restrict__ vks, const int* __restrict__ plists,
                                                cplx* __restrict__ out, int64_t sout, int64_t ldo) {
    const int64_t q = blockIdx.y;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= wp * wp) return;
    const int i = vks[q * wp + e % wp], j = plists[q * wp + e / wp];
    if (i >= 0 && i < w && j < w) out[q * sout + i * ldo + j] = Ms[q * wp * wp + e];
}

// Leaves: M of boundary p alone, [[I, V(b rows of p)], [W(t rows of p), I]]^{-1}, into the
// diagonal block p of R^{-1}.  One workgroup per boundary.
__global__ __launch_bounds__(256) void k_merge_leaf(int64_t nr, int kl, int ku, int64_t bs, int64_t n16,
                                                           const cplx* __restrict__ V, const cplx* __restrict__ W,
                                                           cplx* __restrict__ Rinv, int* __restrict__ info) {
    __shared__ cplx colb[2][kLdsMaxW], rowb[kLdsMaxW];
    __shared__ int plist[kLdsMaxW];
    const int w = kl + ku;
    const int64_t p = blockIdx.x, q = (p + 1) * bs;
    const int r = threadIdx.x % kLdsMaxW, g = threadIdx.x / kLdsMaxW;
    cplx a[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        const int j = 16 * g + c;
        cplx v = mk(r == j ? 1.0 : 0.0, 0.0);
        if (r < kl && j >= kl && j < w) v = V[q - kl + r + (int64_t)(j - kl) * n16];
        if (r >= kl && r < w && j < kl) v = W[q + (r - kl) + (int64_t)j * n16];
        a[c] = v;
    }
    int vk;
    if (!gauss_jordan(a, w, colb, rowb, plist, vk)) {
        if (threadIdx.x == 0) *info = 1;
        return;
    }
    if (r < w) {
        cplx* out = Rinv + (p * w + vk) * nr + p * w;
#pragma unroll
        for (int c = 0; c < 16; ++c)
            if (16 * g + c < w) out[plist[16 * g + c]] = a[c];
    }
}

// C(r, c) = sum_t A[r lda + t] B(t, c) (B[t + c ldb] with BT, else B[t ldb + c]) at
// C[r ldc + c], r < rows, c < cols, t < inner: a 64 x 64 tile per workgroup, 4 x 4 entries a
// thread, 16 terms at a time through LDS, each entry's terms in ascending order.
template <bool BT>
__device__ __forceinline__ void merge_tile(int64_t rows, int row_tile, int64_t cols, int inner, const cplx* A,
                                           int64_t lda, const cplx* B, int64_t ldb, cplx* C, int64_t ldc) {
    __shared__ cplx As[64][17], Bs[64][17];
    const int64_t c0 = (int64_t)blockIdx.x * 64, r0 = (int64_t)row_tile * 64;
    if (c0 >= cols || r0 >= rows) return;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    cplx acc[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[u][v] = mk(0.0, 0.0);
    for (int t0 = 0; t0 < inner; t0 += 16) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int e = (int)threadIdx.x + 256 * k;
            const int ta = e & 15, ra = e >> 4;
            As[ra][ta] = (t0 + ta < inner && r0 + ra < rows) ? A[(r0 + ra) * lda + t0 + ta] : mk(0.0, 0.0);
            const int tb = BT ? (e & 15) : (e >> 6), cb = BT ? (e >> 4) : (e & 63);
            cplx v = mk(0.0, 0.0);
            if (t0 + tb < inner && c0 + cb < cols) v = BT ? B[t0 + tb + (c0 + cb) * ldb] : B[(t0 + tb) * ldb + c0 + cb];
            Bs[cb][tb] = v;
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            cplx a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) a[u] = As[ty + 16 * u][t];
#pragma unroll
            for (int v = 0; v < 4; ++v) b[v] = Bs[tx + 16 * v][t];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = fma_c(acc[u][v], a[u], b[v]);
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t r = r0 + ty + 16 * u, c = c0 + tx + 16 * v;
            if (r < rows && c < cols) C[r * ldc + c] = acc[u][v];
        }
}

// Pair q of a merge: boundaries [a0, a0 + u1) and [a0 + u1, a0 + u1 + u2), a0 = first + q
// stride, m = (u1 + u2) w.  Pt(k, i) = P(i, k) (w x m, column-major), its two blocks that are
// not zero (blockIdx.z = 2 q + block).  One entry per thread, gathered column by column, took
// 0.56 ms a level at w = 400, nr = 4,000.
__global__ __launch_bounds__(256) void k_merge_p(int64_t nr, int kl, int ku, int64_t bs, int64_t n16,
                                                 const cplx* __restrict__ V, const cplx* __restrict__ W,
                                                 const cplx* __restrict__ Rinv, int64_t first, int64_t stride,
                                                 int64_t u1, int64_t u2, cplx* __restrict__ Pt) {
    const int w = kl + ku;
    const int64_t q = blockIdx.z >> 1, a0 = first + q * stride, m1 = u1 * w, m = m1 + u2 * w;
    const cplx* M = Rinv + a0 * w * nr + a0 * w;
    cplx* P = Pt + q * m * w;
    const bool second = (blockIdx.z & 1) != 0;
    // M1[i, t of the last boundary] E, E = V(t rows of that boundary); M2[i, b of the first
    // boundary] F, F = W(b rows of that boundary)
    merge_tile<true>(second ? m - m1 : m1, (int)blockIdx.y, second ? kl : ku, second ? kl : ku,
                     second ? M + m1 * nr + m1 : M + (u1 - 1) * w + kl, nr,
                     second ? W + (a0 + u1 + 1) * bs - kl : V + (a0 + u1) * bs, n16, second ? P + m1 * w : P + kl, w);
}

// S^{-1} of every pair (w x w, by rows), S from the rows of P at beta and alpha.
__global__ __launch_bounds__(256) void k_merge_s(int kl, int ku, int64_t u1, int64_t u2,
                                                        const cplx* __restrict__ Pt, cplx* __restrict__ Sinv,
                                                        int* __restrict__ info) {
    __shared__ cplx colb[2][kLdsMaxW], rowb[kLdsMaxW];
    __shared__ int plist[kLdsMaxW];
    const int w = kl + ku;
    const int64_t m1 = u1 * w, m = m1 + u2 * w;
    const cplx* P = Pt + (int64_t)blockIdx.x * m * w;
    const int r = threadIdx.x % kLdsMaxW, g = threadIdx.x / kLdsMaxW;
    cplx a[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        const int j = 16 * g + c;
        cplx v = mk(r == j ? 1.0 : 0.0, 0.0);
        if (r < kl && j >= kl && j < w) v = P[j + (m1 - w + r) * w];        // row beta_r: (M1[:, t] E)[b_r]
        if (r >= kl && r < w && j < kl) v = P[j + (m1 + r) * w];            // row alpha: (M2[:, b] F)[t]
        a[c] = v;
    }
    int vk;
    if (!gauss_jordan(a, w, colb, rowb, plist, vk)) {
        if (threadIdx.x == 0) *info = 1;
        return;
    }
    if (r < w) {
        cplx* out = Sinv + (int64_t)blockIdx.x * w * w + (int64_t)vk * w;
#pragma unroll
        for (int c = 0; c < 16; ++c)
            if (16 * g + c < w) out[plist[16 * g + c]] = a[c];
    }
}

// Zt(j, i) = Z(i, j), Z = S^{-1} Q (m x w, column-major); blockIdx.z = 2 q + range of j.
__global__ __launch_bounds__(256) void k_merge_z(int64_t nr, int kl, int ku, const cplx* __restrict__ Rinv,
                                                 int64_t first, int64_t stride, int64_t u1, int64_t u2,
                                                 const cplx* __restrict__ Sinv, cplx* __restrict__ Zt) {
    const int w = kl + ku;
    const int64_t q = blockIdx.z >> 1, a0 = first + q * stride, m1 = u1 * w, m = m1 + u2 * w;
    const cplx* M = Rinv + a0 * w * nr + a0 * w;
    const cplx* S = Sinv + q * w * w;
    cplx* Z = Zt + q * m * w;
    const bool second = (blockIdx.z & 1) != 0;
    merge_tile<false>(w, (int)blockIdx.y, second ? m - m1 : m1, second ? ku : kl, second ? S + kl : S, w,
                      second ? M + (m1 + kl) * nr + m1 : M + (m1 - w) * nr, nr, second ? Z + m1 : Z, m);
}

// M = diag(M1, M2) - P Z; X (m x m, by rows) = P Z.
__global__ __launch_bounds__(256) void k_merge_update(int64_t nr, int w, int64_t first, int64_t stride, int64_t u1,
                                                      int64_t u2, const cplx* __restrict__ X,
                                                      cplx* __restrict__ Rinv) {
    const int64_t a0 = first + (int64_t)blockIdx.z * stride, m1 = u1 * w, m = m1 + u2 * w;
    const int64_t i = blockIdx.y, j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= m) return;
    cplx* at = Rinv + (a0 * w + i) * nr + a0 * w + j;
    const cplx x = X[((int64_t)blockIdx.z * m + i) * m + j];
    *at = ((i < m1) == (j < m1)) ? *at - x : -x;
}

// Rinv from the spikes by merging; *info (device, zero on entry) set if a small system is
// singular.  The scratch is freed in st's order.
simm_status merge_inverse(const SpikeFactor& f, int* info, hipStream_t st) {
    const int kl = f.pkl, ku = f.pku, w = kl + ku;
    const int64_t nb = f.nbk - 1, nr = f.nr, n16 = f.n16;
    // the Gauss-Jordan steps' matrices and their pivots (wider couplings)
    const int wp = (w + 15) / 16 * 16;
    struct Free {
        void* q;
        hipStream_t st;
        ~Free() {
            device_free_ordered(q, st);
        }
    } gj{nullptr, st}, fr{nullptr, st};
    cplx* Ms = nullptr;
    int *vks = nullptr, *plists = nullptr;
    if (w > kLdsMaxW) {
        const size_t mats = sizeof(cplx) * (size_t)nb * wp * wp;
        SIMM_HIP_TRY(device_malloc_ordered(&gj.q, mats + 2 * sizeof(int) * (size_t)nb * wp, st));
        Ms = reinterpret_cast<cplx*>(gj.q);
        vks = reinterpret_cast<int*>(static_cast<char*>(gj.q) + mats);
        plists = vks + nb * wp;
    }
    const unsigned gw = (unsigned)((wp * wp + 255) / 256);
    auto gj_inverse = [&](int64_t count, cplx* out, int64_t sout, int64_t ldo) {
        const dim3 grid((unsigned)(1 + wp / 4), (unsigned)count);
        for (int b = -1; b < wp / 16; ++b) {
            const dim3 g = b < 0 ? dim3(1, (unsigned)count) : grid;
            if (wp <= 128) hipLaunchKernelGGL(k_gj_step<128>, g, dim3(128), 0, st, wp, b, Ms, vks, plists, info);
            else if (wp <= 256) hipLaunchKernelGGL(k_gj_step<256>, g, dim3(256), 0, st, wp, b, Ms, vks, plists, info);
            else hipLaunchKernelGGL(k_gj_step<512>, g, dim3(512), 0, st, wp, b, Ms, vks, plists, info);
        }
        hipLaunchKernelGGL(k_gj_out, dim3(gw, (unsigned)count), dim3(256), 0, st, w, wp, (const cplx*)Ms,
                           (const int*)vks, (const int*)plists, out, sout, ldo);
    };
    if (w <= kLdsMaxW) {
        hipLaunchKernelGGL(k_merge_leaf, dim3((unsigned)nb), dim3(256), 0, st, nr, kl, ku, f.bs, f.n16,
                           (const cplx*)f.Vs, (const cplx*)f.Ws, f.Rinv, info);
    } else {
        hipLaunchKernelGGL(k_gj_fill, dim3(gw, (unsigned)nb), dim3(256), 0, st, w, kl, wp,
                           (const cplx*)f.Vs + f.bs - kl, f.bs, (int64_t)1, n16, (const cplx*)f.Ws + f.bs, f.bs,
                           (int64_t)1, n16, Ms, vks);
        gj_inverse(nb, f.Rinv, w * nr + w, nr);
    }
    SIMM_HIP_TRY(hipGetLastError());
    if (nb == 1) return SIMM_OK;
    // scratch of the widest level: P and Z of all pairs (nr w each), S^{-1} of at most nb / 2
    // pairs, and the products of the last level (nr^2)
    void* mem = nullptr;
    const size_t pz = (size_t)nr * w, ss = (size_t)(nb / 2 + 1) * w * w;
    SIMM_HIP_TRY(device_malloc_ordered(&mem, sizeof(cplx) * (2 * pz + ss + (size_t)nr * nr), st));
    fr.q = mem;
    cplx* Pt = reinterpret_cast<cplx*>(mem);
    cplx* Zt = Pt + pz;
    cplx* Sinv = Zt + pz;
    cplx* X = Sinv + ss;
    auto merge = [&](int64_t first, int64_t stride, int64_t u1, int64_t u2, int64_t pairs) -> simm_status {
        const int64_t m = (u1 + u2) * w;
        const unsigned np = (unsigned)pairs, tw = (unsigned)((w + 63) / 64);
        const int64_t m1 = u1 * w, m2 = u2 * w;
        const unsigned tm = (unsigned)((std::max(m1, m2) + 63) / 64);
        hipLaunchKernelGGL(k_merge_p, dim3((unsigned)((std::max(kl, ku) + 63) / 64), tm, 2 * np), dim3(256), 0, st, nr,
                           kl, ku, f.bs, f.n16, (const cplx*)f.Vs, (const cplx*)f.Ws, (const cplx*)f.Rinv, first,
                           stride, u1, u2, Pt);
        if (w <= kLdsMaxW) {
            hipLaunchKernelGGL(k_merge_s, dim3(np), dim3(256), 0, st, kl, ku, u1, u2, (const cplx*)Pt, Sinv, info);
        } else {
            // S from the rows of P at beta and alpha, as in k_merge_s
            hipLaunchKernelGGL(k_gj_fill, dim3(gw, np), dim3(256), 0, st, w, kl, wp,
                               (const cplx*)Pt + kl + (u1 * w - w) * w, m * w, (int64_t)w, (int64_t)1,
                               (const cplx*)Pt + (u1 * w + kl) * w, m * w, (int64_t)w, (int64_t)1, Ms, vks);
            gj_inverse(pairs, Sinv, (int64_t)w * w, w);
        }
        hipLaunchKernelGGL(k_merge_z, dim3(tm, tw, 2 * np), dim3(256), 0, st, nr, kl, ku, (const cplx*)f.Rinv, first,
                           stride, u1, u2, (const cplx*)Sinv, Zt);
        // X^T = Zt Pt (column-major), i.e. P Z by rows: rows of the first range with the last ku
        // columns of P, those of the second with its first kl (the others are zero)
        SIMM_TRY(project_batched(m, ku, Zt + kl * m, m, m * w, Pt + kl, w, m * w, m1, X, m * m, (int)pairs, st));
        SIMM_TRY(project_batched(m, kl, Zt, m, m * w, Pt + m1 * w, w, m * w, m2, X + m1 * m, m * m, (int)pairs, st));
        hipLaunchKernelGGL(k_merge_update, dim3((unsigned)((m + 255) / 256), (unsigned)m, np), dim3(256), 0, st, nr, w,
                           first, stride, u1, u2, (const cplx*)X, f.Rinv);
        SIMM_HIP_TRY(hipGetLastError());
        return SIMM_OK;
    };
    for (int64_t u = 1; u < nb; u *= 2) {
        const int64_t full = nb / (2 * u), rem = nb - full * 2 * u;
        if (full > 0) SIMM_TRY(merge(0, 2 * u, u, u, full));
        if (rem > u) SIMM_TRY(merge(full * 2 * u, 0, u, rem - u, 1));
    }
    return SIMM_OK;
}

// z_i = sum_c Rinv[i, c] g[tip(c)] for NR right-hand sides (g + r ldg -> z + r ldz): one
// wavefront per reduced row, four accumulators per lane and column (a column's
// operations are those of NR = 1).  Bound by the read of Rinv.  The tips are gathered once
// per workgroup of 8 rows, 1,024 at a time, while the first 16 loads of each row are on
// their way: 10.7 us at nr = 1,568 (3.7 TB/s), 3.9 us at 224; gathered by every row, with a
// 64-bit division per entry, it took 22.8 and 9.3 us.
constexpr int kTipTile = 1024;
template <int NR>
__global__ __launch_bounds__(512) void k_part_tips(int nr, int kl, int ku, int64_t bs,
                                                   const cplx* __restrict__ Rinv, const cplx* __restrict__ g,
                                                   int64_t ldg, cplx* __restrict__ z, int64_t ldz,
                                                   const int* active) {
    if (active && *active == 0) return;
    extern __shared__ double2 zsm[];
    cplx* gs = reinterpret_cast<cplx*>(zsm);   // NR x min(nr, kTipTile)
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 8 + (threadIdx.x >> 6);
    const cplx* row = Rinv + (int64_t)min(i, nr - 1) * nr;
    const int ld = min(nr, kTipTile), w = kl + ku;
    cplx acc[NR][4];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[r][u] = mk(0.0, 0.0);
    for (int t0 = 0; t0 < nr; t0 += kTipTile) {
        const int cnt = min(kTipTile, nr - t0);
        cplx rv[16];
#pragma unroll
        for (int h = 0; h < 4; ++h)
            if (256 * h < cnt) {
#pragma unroll
                for (int u = 0; u < 4; ++u) rv[4 * h + u] = row[t0 + min(256 * h + 64 * u + lane, cnt - 1)];
            }
        if (t0 > 0) __syncthreads();
        for (int e = threadIdx.x; e < cnt; e += 512) {
            const unsigned c = (unsigned)(t0 + e), p = c / (unsigned)w;
            const int r = (int)(c - p * (unsigned)w);
            const int64_t tr = (int64_t)(p + 1) * bs + (r - kl);   // b_p (r < kl), then t_{p+1}
#pragma unroll
            for (int v = 0; v < NR; ++v) gs[v * ld + e] = g[tr + v * ldg];
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 4; ++h)
            if (256 * h < cnt) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = 256 * h + 64 * u + lane;
                    if (e < cnt) {
#pragma unroll
                        for (int r = 0; r < NR; ++r) acc[r][u] = fma_c(acc[r][u], rv[4 * h + u], gs[r * ld + e]);
                    }
                }
            }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        cplx t = (acc[r][0] + acc[r][1]) + (acc[r][2] + acc[r][3]);
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            t.re += __shfl_xor(t.re, m, 64);
            t.im += __shfl_xor(t.im, m, 64);
        }
        if (lane == 0 && i < nr) z[i + r * ldz] = t;
    }
}

// y_i = g_i - sum_k V[i,k] t_j[k] - sum_k W[i,k] b_{j-1}[k], j the block of row i: 64 rows
// per workgroup, the tips of their (at most two) blocks staged in LDS, wavefront q taking
// the terms k = q mod 4 of each sum; NR right-hand sides (z + r ldz, g + r ldg, y + r ldy)
// share the loads of V and W.  Bound by that read; the first loads leave before the tips
// are staged.  4.6 us at n = 14,167, w = 32 (8.5 us with 256 rows per workgroup, one thread
// each: 56 workgroups); at n = 250,000, w = 128 88 us, 5.8 TB/s.
template <int NR>
__global__ __launch_bounds__(256) void k_part_correct(int64_t n, int64_t n16, int kl, int ku, int64_t bs,
                                                      int64_t nbk, const cplx* __restrict__ V,
                                                      const cplx* __restrict__ W, const cplx* __restrict__ z,
                                                      int64_t ldz, const cplx* __restrict__ g, int64_t ldg,
                                                      cplx* __restrict__ y, int64_t ldy, const int* active) {
    if (active && *active == 0) return;
    extern __shared__ double2 zsm[];
    // NR x 2 x (ku + kl): t_j then b_{j-1}, for blocks jb, jb + 1; then the wavefronts' sums
    cplx* zs = reinterpret_cast<cplx*>(zsm);
    const int w = kl + ku;
    cplx* part = zs + NR * 2 * w;                       // NR x 3 x 64
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int64_t jb = r0 / bs;
    const int64_t i = min(r0 + lane, n - 1);
    cplx v0[8], w0[4];
#pragma unroll
    for (int u = 0; u < 8; ++u)
        if (4 * u + wv < ku) v0[u] = V[i + (int64_t)(4 * u + wv) * n16];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (4 * u + wv < kl) w0[u] = W[i + (int64_t)(4 * u + wv) * n16];
    for (int e = threadIdx.x; e < 2 * w; e += 256) {
        const int64_t j = jb + e / w;
        const int q = e % w;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            cplx v = mk(0.0, 0.0);
            if (q < ku) {
                if (j <= nbk - 2) v = z[j * w + kl + q + r * ldz];
            } else {
                if (j >= 1 && j <= nbk - 1) v = z[(j - 1) * w + (q - ku) + r * ldz];
            }
            zs[r * 2 * w + e] = v;
        }
    }
    __syncthreads();
    const int64_t j = i / bs;
    const int off = (int)(j - jb) * w;          // t_j (ku values), then b_{j-1} (kl values)
    cplx acc[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r] = mk(0.0, 0.0);
    auto term = [&](cplx v, int k) {
#pragma unroll
        for (int r = 0; r < NR; ++r) acc[r] = fma_c(acc[r], v, zs[r * 2 * w + off + k]);
    };
    if (j <= nbk - 2) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (4 * u + wv < ku) term(v0[u], 4 * u + wv);
#pragma unroll 8
        for (int k = 32 + wv; k < ku; k += 4) term(V[i + (int64_t)k * n16], k);
    }
    if (j >= 1) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (4 * u + wv < kl) term(w0[u], ku + 4 * u + wv);
#pragma unroll 8
        for (int k = 16 + wv; k < kl; k += 4) term(W[i + (int64_t)k * n16], ku + k);
    }
    if (wv > 0) {
#pragma unroll
        for (int r = 0; r < NR; ++r) part[(r * 3 + wv - 1) * 64 + lane] = acc[r];
    }
    __syncthreads();
    if (wv > 0 || r0 + lane >= n) return;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const cplx* pr = part + r * 3 * 64 + lane;
        y[i + r * ldy] = g[i + r * ldg] - ((acc[r] + pr[0]) + (pr[64] + pr[128]));
    }
}

// V and W: D^{-1} of all kl + ku coupling columns, in place (Vs and Ws are one n16 x
// (kl + ku) array), the columns in the same launches.  (Four columns a launch, dealt to four
// streams, left the device waiting on launches and chains: n = 250,000 27.8 -> 23.9 ms,
// n = 100,000 5.3 -> 3.3 ms.)
simm_status spikes(const SpikeFactor& f, hipStream_t st) {
    const int kl = f.pkl, ku = f.pku, w = kl + ku;
    const int64_t n16 = f.n16;
    SpikeFactor cl;
    // (freed in st's order: a plain free would wait for the whole device)
    // scratch of all columns, which is as much as the spikes themselves; of fewer at a time where
    // memory does not hold it
    int cols = f.cbs > 0 ? w : spike_max_nrhs(f);
    for (;;) {
        const simm_status rc = spike_clone_scratch(f, cl, st, cols, true);
        if (rc == SIMM_OK) break;
        if (rc != SIMM_ENOMEM || cols == 1) return rc;
        cols = (cols + 1) / 2;
    }
    struct Release {
        SpikeFactor* c;
        hipStream_t st;
        ~Release() { spike_release_ordered(*c, st); }
    } rel{&cl, st};
    ChainSlots slots;   // (chains only without chunks inside blocks; released after a synchronize)
    SIMM_TRY(slots.acquire(spike_chain_weight(f), st));
    hipLaunchKernelGGL(k_part_rhs, dim3((unsigned)((n16 + 255) / 256), (unsigned)w), dim3(256), 0, st, f.n, n16, kl, ku,
                       f.bs, f.nbk, f.cpl, f.Vs);
    SIMM_HIP_TRY(hipGetLastError());
    SIMM_TRY(spike_apply_diag_cols(cl, f.Vs, w, st));
    if (f.cbs > 0) return SIMM_OK;
    int err = 0;
    SIMM_HIP_TRY(hipMemcpyAsync(&err, cl.err, sizeof(int), hipMemcpyDeviceToHost, st));
    SIMM_HIP_TRY(hipStreamSynchronize(st));
    if (err) {
        set_error("partitioned factorization: a chunk-chain barrier of a spike solve timed out");
        return SIMM_EHIP;
    }
    return SIMM_OK;
}

template <typename CT>
simm_status cut_t(int64_t n, int kl, int ku, CT* AB, int64_t bs, cplx* cpl, hipStream_t st) {
    const int64_t nbk = (n + bs - 1) / bs;
    if (nbk < 2) return SIMM_OK;
    hipLaunchKernelGGL(k_part_cut<CT>, dim3((unsigned)(nbk - 1)), dim3(256), 0, st, n, kl, ku, AB, bs, cpl);
    SIMM_HIP_TRY(hipGetLastError());
    return SIMM_OK;
}

}  // namespace

simm_status part_cut(int64_t n, int kl, int ku, cplx* AB, int64_t bs, cplx* cpl, hipStream_t st) {
    return cut_t(n, kl, ku, AB, bs, cpl, st);
}
simm_status part_cut(int64_t n, int kl, int ku, cplxf* AB, int64_t bs, cplx* cpl, hipStream_t st) {
    return cut_t(n, kl, ku, AB, bs, cpl, st);
}

size_t part_prepare_bytes(int64_t n, int kl, int ku, int64_t bs, size_t spike_scratch) {
    const size_t n16 = (size_t)((n + 15) / 16 * 16), w = (size_t)(kl + ku), nb = (size_t)((n + bs - 1) / bs) - 1;
    const size_t nr = nb * w;
    const size_t merge = sizeof(cplx) * (2 * nr * w + (nb / 2 + 1) * w * w + nr * nr);
    return sizeof(cplx) * (n16 * w + nr * nr + n16 + nr) + std::max(spike_scratch, merge);
}

simm_status part_prepare(SpikeFactor& f, hipStream_t st) {
    const int kl = f.kl, ku = f.ku, w = kl + ku;
    f.pkl = kl;
    f.pku = ku;
    f.nbk = (f.n + f.bs - 1) / f.bs;
    f.nr = (f.nbk - 1) * (int64_t)w;
    const int64_t n16 = f.n16, nr = f.nr;
    if (f.nbk < 2 || nr > kPartMaxReduced || w > kMergeMaxW) {
        set_error("partitioned factorization: block layout out of range");
        return SIMM_EUNSUPPORTED;
    }
    const size_t elems = (size_t)n16 * w + (size_t)nr * nr + (size_t)n16 + (size_t)nr + 64;
    SIMM_HIP_TRY(device_malloc(&f.part_mem, sizeof(cplx) * elems + 8 * 256));
    char* p = reinterpret_cast<char*>(f.part_mem);
    auto take = [&](size_t count) {
        char* r = p;
        p += (sizeof(cplx) * count + 255) & ~(size_t)255;
        return reinterpret_cast<cplx*>(r);
    };
    f.Vs = take((size_t)n16 * w);          // (n16 is a multiple of 16: the columns of W follow V's)
    f.Ws = f.Vs + (size_t)n16 * ku;
    f.Rinv = take((size_t)nr * nr);
    f.pg = take((size_t)n16);
    f.pz = take((size_t)nr);
    // SIMM_PART_TIMING: the phases' times on stderr
    const bool timing = getenv("SIMM_PART_TIMING") != nullptr;
    const auto t0 = std::chrono::steady_clock::now();
    auto stamp = [&](const char* what, std::chrono::steady_clock::time_point& since) {
        if (!timing) return;
        (void)hipStreamSynchronize(st);
        const auto now = std::chrono::steady_clock::now();
        std::fprintf(stderr, "[simm part] n = %lld, %lld blocks of %lld: %s %.2f ms\n", (long long)f.n,
                     (long long)f.nbk, (long long)f.bs, what,
                     std::chrono::duration<double, std::milli>(now - since).count());
        since = now;
    };
    auto tp = t0;
    SIMM_TRY(spikes(f, st));
    stamp("spikes", tp);
    int* info = nullptr;
    SIMM_HIP_TRY(device_malloc_ordered((void**)&info, sizeof(int), st));
    struct FreeInfo {
        void* q;
        hipStream_t st;
        ~FreeInfo() { device_free_ordered(q, st); }
    } fi{info, st};
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, info, 0);
    SIMM_TRY(merge_inverse(f, info, st));
    int singular = 0;
    SIMM_HIP_TRY(hipMemcpyAsync(&singular, info, sizeof(int), hipMemcpyDeviceToHost, st));
    SIMM_HIP_TRY(hipStreamSynchronize(st));
    stamp("reduced inverse", tp);
    if (singular) {
        set_error("partitioned factorization: the reduced system is singular");
        return SIMM_ESINGULAR_SHIFT;
    }
    return SIMM_OK;
}

namespace {
template <int NR>
void part_tail(const SpikeFactor& f, cplx* y, int64_t ldy, const int* active, hipStream_t st) {
    hipLaunchKernelGGL((k_part_tips<NR>), dim3((unsigned)((f.nr + 7) / 8)), dim3(512),
                       sizeof(cplx) * NR * (size_t)std::min<int64_t>(f.nr, kTipTile), st, (int)f.nr, f.pkl, f.pku, f.bs,
                       (const cplx*)f.Rinv, (const cplx*)f.pg, f.n16, f.pz, f.nr, active);
    hipLaunchKernelGGL((k_part_correct<NR>), dim3((unsigned)((f.n + 63) / 64)), dim3(256),
                       sizeof(cplx) * (2 * (size_t)(f.pkl + f.pku) + 3 * 64) * NR, st, f.n, f.n16, f.pkl, f.pku, f.bs, f.nbk,
                       (const cplx*)f.Vs, (const cplx*)f.Ws, (const cplx*)f.pz, f.nr, (const cplx*)f.pg, f.n16, y, ldy,
                       active);
}
}  // namespace

simm_status part_apply(const SpikeFactor& f, const cplx* u, cplx* y, const int* active, hipStream_t st) {
    SIMM_TRY(spike_apply_diag(f, u, f.pg, active, st));
    part_tail<1>(f, y, f.n16, active, st);
    SIMM_HIP_TRY(hipGetLastError());
    return SIMM_OK;
}

simm_status part_apply_nr(const SpikeFactor& f, const cplx* u, int64_t ldu, cplx* y, int64_t ldy, int nr,
                          hipStream_t st) {
    // g = D^{-1} u for the nr columns (f.pg and f.pz hold f.nrhs columns each)
    SIMM_TRY(spike_apply_diag_nr(f, u, ldu, f.pg, f.n16, nr, st));
    if (nr == 4) part_tail<4>(f, y, ldy, nullptr, st);
    else if (nr == 2) part_tail<2>(f, y, ldy, nullptr, st);
    else part_tail<1>(f, y, ldy, nullptr, st);
    SIMM_HIP_TRY(hipGetLastError());
    return SIMM_OK;
}

}  // namespace simm
