// Arnoldi process of Sec. 2 on M = (A - sigma B)^{-1} B, one column j at a time:
//   w = M v_j;  h_{1:j,j} = V_j^H w;  w -= V_j h;  (repeated once: classical
//   Gram-Schmidt applied twice);  h_{j+1,j} = ||w||;  v_{j+1} = w / h_{j+1,j};
// with the happy-breakdown stop h_{j+1,j} <= 1e-14 ||M v_j||.
//
// Reductions over the n rows are two-stage and in a fixed order (per-block partial
// sums, then one block summing the partials sequentially), so every run gives
// bitwise the same H.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace simm {

namespace {

constexpr int GS_WAVES = 8;
constexpr int GS_THREADS = 64 * GS_WAVES;

// Sums over the wavefront of N (a power of two, at most 64) values a lane: halving
// exchanges, so that N values take about N lane exchanges instead of 6 N; lane l returns
// the sum of value l / (64 / N).
template <int N>
__device__ __forceinline__ cplx wave_sums(cplx (&v)[N], int lane) {
    if constexpr (N == 1) {
        cplx t = v[0];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) t = t + mk(__shfl_xor(t.re, m, 64), __shfl_xor(t.im, m, 64));
        return t;
    } else {
#pragma unroll
        for (int half = N / 2, m = 32; half >= 1; half >>= 1, m >>= 1) {
            const bool up = (lane & m) != 0;
#pragma unroll
            for (int i = 0; i < half; ++i) {
                const cplx send = csel(up, v[i], v[i + half]);
                const cplx keep = csel(up, v[i + half], v[i]);
                v[i] = keep + mk(__shfl_xor(send.re, m, 64), __shfl_xor(send.im, m, 64));
            }
        }
        cplx t = v[0];
#pragma unroll
        for (int m = 32 / N; m >= 1; m >>= 1) t = t + mk(__shfl_xor(t.re, m, 64), __shfl_xor(t.im, m, 64));
        return t;
    }
}

constexpr int pow2_at_least(int q) { return q <= 1 ? 1 : q <= 2 ? 2 : q <= 4 ? 4 : q <= 8 ? 8 : 16; }

// One pass over the first ncol columns of V for the block's rows (chunks of 64, a row a
// lane; wavefront v takes columns v, v + 8, ..., at most NQ of them):
//   UPD:  w -= V h (the wavefronts' shares meet in LDS, summed in their order);
//   DOTS: partial sums of conj(V(r, i)) w(r), i < ncol, on the updated rows;
//   NORM: of |w(r)|^2 (column ncol, or 0 without DOTS).
// h comes from the reduction kernel, or (h null) from the previous pass's partial sums
// `hpart`, which every workgroup then adds up for itself and the first leaves in hout.
// A pass reads V once: the entries that form the update stay in registers for the sums.
// (They were read again for the sums, and the sums took a 6-step lane reduction per column
// and 64 rows.  n = 250,000, m = 120: 195 us a step on average for the three passes, now 137,
// 5.2 TB/s at 106 columns; n = 400, m = 40: 22 us, now 12.)  partial[i nblk + blk].
template <int NQ, bool UPD, bool DOTS, bool NORM>
__device__ __forceinline__ void gs_pass(int64_t n, const cplx* __restrict__ V, int64_t ldv, int ncol,
                                        const cplx* __restrict__ h, const cplx* __restrict__ hpart,
                                        cplx* __restrict__ hout, cplx* __restrict__ w, cplx* __restrict__ partial,
                                        cplx* hs, cplx (*part)[GS_WAVES][64]) {
    constexpr int N = pow2_at_least(NQ);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t nblk = gridDim.x, chunks = (n + 63) / 64, per = (chunks + nblk - 1) / nblk;
    const int64_t k0 = blockIdx.x * per, k1 = min(chunks, k0 + per);
    if constexpr (UPD) {
        if (h != nullptr) {
            for (int i = threadIdx.x; i < GS_WAVES * NQ; i += GS_THREADS) hs[i] = i < ncol ? h[i] : mk(0.0, 0.0);
        } else {
            cplx s[N];
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const int i = wave + GS_WAVES * q;
                s[q] = mk(0.0, 0.0);
                if (i < ncol && lane < nblk) s[q] = hpart[i * nblk + lane];   // nblk <= 64
            }
            const cplx t = wave_sums<N>(s, lane);
            const int q = lane / (64 / N);
            if (lane % (64 / N) == 0 && q < NQ) {
                hs[wave + GS_WAVES * q] = t;
                if (blockIdx.x == 0 && wave + GS_WAVES * q < ncol) hout[wave + GS_WAVES * q] = t;
            }
        }
        __syncthreads();
    }
    cplx acc[DOTS ? NQ : 1];
#pragma unroll
    for (int q = 0; q < (DOTS ? NQ : 1); ++q) acc[q] = mk(0.0, 0.0);
    double nrm = 0.0;
    for (int64_t k = k0; k < k1; ++k) {
        const int64_t r = k * 64 + lane, rc = min(r, n - 1);
        cplx v[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[q] = V[rc + (int64_t)min(wave + GS_WAVES * q, ncol - 1) * ldv];
        cplx x = mk(0.0, 0.0);
        // (updates: only the wavefront that writes w reads it)
        if (!UPD || wave == 0) x = w[rc];
        if constexpr (UPD) {
            cplx p = x;
#pragma unroll
            for (int q = 0; q < NQ; ++q) p = fms(p, v[q], hs[wave + GS_WAVES * q]);
            cplx(*pt)[64] = part[k & 1];
            pt[wave][lane] = p;
            lds_barrier();
            x = pt[0][lane];
#pragma unroll
            for (int u = 1; u < GS_WAVES; ++u) x = x + pt[u][lane];
            if (wave == 0 && r < n) w[r] = x;
        }
        if (r >= n) x = mk(0.0, 0.0);
        if constexpr (DOTS) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q] = fma_cj(acc[q], v[q], x);
        }
        if constexpr (NORM) nrm += norm2(x);
    }
    if constexpr (DOTS) {
        cplx s[N];
#pragma unroll
        for (int q = 0; q < N; ++q) s[q] = q < NQ ? acc[q < NQ ? q : 0] : mk(0.0, 0.0);
        const cplx t = wave_sums<N>(s, lane);
        const int i = wave + GS_WAVES * (lane / (64 / N));
        if (lane % (64 / N) == 0 && i < ncol && lane / (64 / N) < NQ) partial[i * nblk + blockIdx.x] = t;
    }
    if constexpr (NORM) {
        if (wave == 0) {
            cplx s[1] = {mk(nrm, 0.0)};
            const cplx t = wave_sums<1>(s, lane);
            if (lane == 0) partial[(DOTS ? ncol : 0) * nblk + blockIdx.x] = t;
        }
    }
}

// sum of |w(r)|^2 alone (the start vector)
__device__ __forceinline__ void gs_norm_only(int64_t n, const cplx* __restrict__ w, cplx* __restrict__ partial) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t nblk = gridDim.x, chunks = (n + 63) / 64, per = (chunks + nblk - 1) / nblk;
    const int64_t k0 = blockIdx.x * per, k1 = min(chunks, k0 + per);
    double nrm = 0.0;
    if (wave == 0)
        for (int64_t k = k0; k < k1; ++k) {
            const int64_t r = k * 64 + lane;
            if (r < n) nrm += norm2(w[r]);
        }
    if (wave == 0) {
        cplx s[1] = {mk(nrm, 0.0)};
        const cplx t = wave_sums<1>(s, lane);
        if (lane == 0) partial[blockIdx.x] = t;
    }
}

}  // namespace

// The passes of up to four independent Arnoldi processes at once (same n, j and layout;
// space blockIdx.y).  PASS 1: DOTS and NORM, 2: UPD and DOTS, 3: UPD and NORM; self: the
// passes add up the partial sums themselves (up to 64 row blocks).
template <int NQ, int PASS>
__global__ __launch_bounds__(GS_THREADS) void k_gs_pass(int64_t n, GsBatch b, int64_t ldv, int ncol, int self) {
    const int y = blockIdx.y;
    if (*b.active[y] == 0) return;
    __shared__ cplx hs[GS_WAVES * NQ];
    __shared__ cplx part[2][GS_WAVES][64];
    // the sums of passes 1 and 3 go to partial, those of pass 2 to partial2
    cplx* hv = PASS == 2 ? b.h1[y] : b.h2[y];
    gs_pass<NQ, PASS != 1, PASS != 3, PASS != 2>(n, b.V[y], ldv, ncol, self ? nullptr : hv,
                                                 PASS == 2 ? b.partial[y] : b.partial2[y], hv, b.w[y],
                                                 PASS == 2 ? b.partial2[y] : b.partial[y], hs, part);
}

__global__ __launch_bounds__(GS_THREADS) void k_gs_norm(int64_t n, GsBatch b) {
    gs_norm_only(n, b.w[blockIdx.y], b.partial[blockIdx.y]);
}

// out[i] = sum_blk partial[i nblk + blk] for i < ntot: one block per column, a
// fixed-shape tree over the row blocks, so the order never changes.
__device__ __forceinline__ cplx gs_sum_blocks(const cplx* __restrict__ p, int nblk, cplx* red) {
    cplx acc = mk(0.0, 0.0);
    for (int b = threadIdx.x; b < nblk; b += 256) acc = acc + p[b];
    cplx s[1] = {acc};
    const cplx t = wave_sums<1>(s, threadIdx.x & 63);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(256) void k_gs_reduce(GsBatch b, int nblk, int which) {
    const int y = blockIdx.y;
    if (*b.active[y] == 0) return;
    __shared__ cplx red[4];
    const cplx* p = which == 1 ? b.partial[y] : b.partial2[y];
    const cplx t = gs_sum_blocks(p + (int64_t)blockIdx.x * nblk, nblk, red);
    if (threadIdx.x == 0) (which == 1 ? b.h1[y] : b.h2[y])[blockIdx.x] = t;
}

// End of step j and input of the next one, in one launch: every workgroup adds up ||w||^2
// (the same sum in the same order), the first leaves H(0..j, j) = h1 + h2, h_{j+1,j} = ||w||
// and the outcome of the breakdown test against ||M v_j||; then v_{j+1} = w / ||w|| and, with
// u, u = B v_{j+1}.  j = -1: the start vector, ||w|| to hnorm[2].
__global__ __launch_bounds__(256) void k_gs_next(int64_t n, GsBatch b, int64_t ldv, int j, int ldh, int nblk, int self,
                                                 const cplx* __restrict__ Bb, int klb, int kub, int want_u) {
    const int y = blockIdx.y;
    // (the first workgroup may clear the flag below while others start: those skip what a
    // breakdown skips anyway)
    if (*b.active[y] == 0) return;
    __shared__ cplx red[2][4];
    const double wn = sqrt(gs_sum_blocks(b.partial[y], nblk, red[0]).re);
    if (j >= 0) {
        const double w0 =
            sqrt(self ? gs_sum_blocks(b.partial[y] + (int64_t)(j + 1) * nblk, nblk, red[1]).re : b.h1[y][j + 1].re);
        const bool stop = wn <= 1e-14 * w0;
        if (blockIdx.x == 0) {
            cplx* H = b.H[y] + (int64_t)j * ldh;
            for (int i = threadIdx.x; i <= j; i += blockDim.x) H[i] = b.h1[y][i] + b.h2[y][i];
            if (threadIdx.x == 0) {
                b.hnorm[y][0] = wn;
                b.hnorm[y][1] = w0;
                H[j + 1] = mk(stop ? 0.0 : wn, 0.0);
                if (stop) {
                    *b.active[y] = 0;
                    *b.m_eff[y] = j + 1;
                }
            }
        }
        if (stop) return;
    } else if (blockIdx.x == 0 && threadIdx.x == 0) {
        b.hnorm[y][2] = wn;
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const cplx* w = b.w[y];
    // (a division, as written in the Arnoldi step)
    auto scaled = [&](int64_t c) { return mk(w[c].re / wn, w[c].im / wn); };
    const cplx vi = scaled(i);
    b.V[y][i + (int64_t)(j + 1) * ldv] = vi;
    if (!want_u) return;
    cplx acc = vi;
    if (Bb != nullptr) {
        const int ldb = klb + kub + 1;
        acc = mk(0.0, 0.0);
        for (int d = -klb; d <= kub; ++d) {
            const int64_t c = i + d;
            if (c < 0 || c >= n) continue;
            acc = fma_c(acc, Bb[(int64_t)(kub - d) + c * ldb], scaled(c));
        }
    }
    b.u[y][i] = acc;
}

// Row blocks of the passes: 64-row chunks dealt evenly to at most `cap` workgroups.
int gs_row_blocks(int64_t n, int64_t cap) {
    const int64_t chunks = (n + 63) / 64, per = (chunks + cap - 1) / cap;
    return (int)((chunks + per - 1) / per);
}

namespace {
// calls f(std::integral_constant<int, NQ>) with the smallest NQ that holds ncol columns
template <typename F>
void with_nq(int ncol, F f) {
    switch ((ncol + GS_WAVES - 1) / GS_WAVES) {
        case 1: f(std::integral_constant<int, 1>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 3: f(std::integral_constant<int, 3>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        case 5: f(std::integral_constant<int, 5>()); break;
        case 6: f(std::integral_constant<int, 6>()); break;
        case 7:
        case 8: f(std::integral_constant<int, 8>()); break;
        case 9:
        case 10: f(std::integral_constant<int, 10>()); break;
        case 11:
        case 12: f(std::integral_constant<int, 12>()); break;
        case 13:
        case 14: f(std::integral_constant<int, 14>()); break;
        default: f(std::integral_constant<int, 16>()); break;
    }
}
}  // namespace

namespace {
// up to so many row blocks the passes add up the partial sums themselves (n <= 4,096: two
// launches fewer a step; every workgroup then reads all of them)
constexpr int GS_SELF_BLOCKS = 64;

// klb + kub from which B v_{j+1} is a launch of its own, by columns: a row's strided walk, with
// a division per entry of v, costs more than the launch (a build of 60 steps at n = 100,000: 24
// off-diagonals 15.5 and 15.2 ms, 32 17.0 and 16.3, 64 25.1 and 22.8; at n = 1,000 6.5 and 6.6,
// 6.6 and 6.7, 7.3 and 7.0).
constexpr int GS_WIDE_B = 32;

simm_status gs_next(int64_t n, const GsBatch& b, int nr, int64_t ldv, int j, int ldh, int nblk, const cplx* Bb, int klb,
                    int kub, bool want_u, hipStream_t st) {
    const bool wide = want_u && Bb != nullptr && klb + kub >= GS_WIDE_B;
    hipLaunchKernelGGL(k_gs_next, dim3((unsigned)((n + 255) / 256), (unsigned)nr), dim3(256), 0, st, n, b, ldv, j, ldh,
                       nblk, nblk <= GS_SELF_BLOCKS ? 1 : 0, Bb, klb, kub, want_u && !wide ? 1 : 0);
    SIMM_HIP_TRY(hipGetLastError());
    for (int r = 0; wide && r < nr; ++r)
        SIMM_TRY(prepare_input(n, b.V[r] + (int64_t)(j + 1) * ldv, Bb, klb, kub, b.u[r], st));
    return SIMM_OK;
}
}  // namespace

// Start of nr <= 4 processes: beta = ||w|| (hnorm[2]), v_1 = w / beta, u = B v_1.
simm_status arnoldi_start(int64_t n, const GsBatch& b, int nr, int64_t ldv, int nblk, const cplx* Bb, int klb, int kub,
                          hipStream_t st) {
    hipLaunchKernelGGL(k_gs_norm, dim3((unsigned)nblk, (unsigned)nr), dim3(GS_THREADS), 0, st, n, b);
    return gs_next(n, b, nr, ldv, -1, 0, nblk, Bb, klb, kub, true, st);
}

// Step j of nr <= 4 processes, w holding M v_j: classical Gram-Schmidt twice, column j of H,
// v_{j+1} and (want_u) u = B v_{j+1}.
simm_status arnoldi_step(int64_t n, const GsBatch& b, int nr, int64_t ldv, int j, int ldh, int nblk, const cplx* Bb,
                         int klb, int kub, bool want_u, hipStream_t st) {
    const int ncol = j + 1;
    const unsigned y = (unsigned)nr;
    const int self = nblk <= GS_SELF_BLOCKS ? 1 : 0;
    with_nq(ncol, [&](auto nq) {
        constexpr int NQ = decltype(nq)::value;
        const dim3 grid((unsigned)nblk, y);
        // pass 1: h1 = V^H w and ||w||^2; 2: w -= V h1 and h2 = V^H w on the new w
        // (re-orthogonalisation); 3: w -= V h2 and ||w||^2
        hipLaunchKernelGGL((k_gs_pass<NQ, 1>), grid, dim3(GS_THREADS), 0, st, n, b, ldv, ncol, self);
        if (!self) hipLaunchKernelGGL(k_gs_reduce, dim3(ncol + 1, y), dim3(256), 0, st, b, nblk, 1);
        hipLaunchKernelGGL((k_gs_pass<NQ, 2>), grid, dim3(GS_THREADS), 0, st, n, b, ldv, ncol, self);
        if (!self) hipLaunchKernelGGL(k_gs_reduce, dim3(ncol, y), dim3(256), 0, st, b, nblk, 2);
        hipLaunchKernelGGL((k_gs_pass<NQ, 3>), grid, dim3(GS_THREADS), 0, st, n, b, ldv, ncol, self);
    });
    return gs_next(n, b, nr, ldv, j, ldh, nblk, Bb, klb, kub, want_u, st);
}

}  // namespace simm
