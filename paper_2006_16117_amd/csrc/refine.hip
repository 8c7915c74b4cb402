// FP64-residual iterative refinement of solves with an FP32 band factor (mixed
// precision).  The Cayley transform of Sec. 2 needs y = (A - sigma B)^{-1} u for every
// application of M (eq. (IMxb)); with the factor L U ~ P (A - sigma B) held in FP32,
//     x_0 = U^{-1} L^{-1} P u,   r_k = u - (A - sigma B) x_k  (FP64, from the FP64 bands),
//     x_{k+1} = x_k + U^{-1} L^{-1} P r_k,
// until the normwise backward error
//     eta_k = ||r_k||_inf / (||A - sigma B||_inf ||x_k||_inf + ||u||_inf)
// is at most the tolerance.  Every step is decided on the device (a flag that the
// next kernels read), so an application never waits for the host; a step that is not
// needed returns at once.  If the tolerance is not met within the allowed steps an
// error flag is raised and the shift is rebuilt with an FP64 factor by the caller.
#include <cmath>
#include <cstring>

#include "common.hpp"
#include "kernels.hpp"

namespace simm {

namespace {

// non-negative doubles order like their bit patterns
__device__ inline unsigned long long atomic_max_nonneg(unsigned long long* p, double v) {
    return atomicMax(p, (unsigned long long)__double_as_longlong(v));
}
__device__ inline double wave_max64(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmax(v, __shfl_xor(v, m, 64));
    return v;
}

}  // namespace

// After a residual: converged (eta <= tol) ends the refinement; otherwise one more
// correction, or, after the last allowed one, the error flag.  Clears the norms.
__device__ void refine_check(RefineState st, double nr, double nx, double nu, double cnorm, double tol, int last) {
    st.norms[0] = st.norms[1] = st.norms[2] = 0ull;
    const double den = cnorm * nx + nu;
    const double eta = den > 0.0 ? nr / den : 0.0;
    if (eta <= tol) {
        st.flags[0] = 0;
        st.stats[0] += 1;                           // applications
        if (eta > __longlong_as_double((long long)st.norms[3])) st.norms[3] = (unsigned long long)__double_as_longlong(eta);
    } else if (last) {
        st.flags[0] = 0;
        st.flags[1] = 1;                            // tolerance not reached
        st.stats[0] += 1;
        if (eta > __longlong_as_double((long long)st.norms[3])) st.norms[3] = (unsigned long long)__double_as_longlong(eta);
    } else {
        st.stats[1] += 1;                           // corrections
    }
}

// r = u - (A - sigma B) x, row by row, and the infinity norms of r, x and u
// (norms[0..2], as the bit patterns of non-negative doubles).  Skipped when *gate == 0.
// A workgroup takes 64 consecutive rows; its wavefronts share the columns that meet them in
// consecutive ranges: at column j the lanes read the entries (i, j) of their rows,
// which are consecutive in band storage (one coalesced load, out-of-band taps clamped into
// the band and dropped; x_j is the same for every lane).  Each row's entries are accumulated
// in ascending column order within a range, the ranges in order.  Bound by the loads in
// flight: one wavefront per 64 rows with four loads ahead took 52 us at n = 20,000,
// kl = ku = 64, four with eight ahead 23 us, eight 19 us.  With st.flags set (a refinement step) the workgroup that adds
// its norms last decides the step (refine_check; norms[5] counts the workgroups).
constexpr int kResidWaves = 8;
__global__ __launch_bounds__(64 * kResidWaves) void k_band_resid(int64_t n, const cplx* __restrict__ A, int kla, int kua,
                                                    const cplx* __restrict__ B, int klb, int kub, cplx sigma,
                                                    const cplx* __restrict__ u, const cplx* __restrict__ x,
                                                    cplx* __restrict__ r, unsigned long long* norms, const int* gate,
                                                    RefineState rs, double cnorm, double tol, int last) {
    if (*gate == 0) return;
    __shared__ cplx part[kResidWaves - 1][64];
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = r0 + lane;
    const int lda = kla + kua + 1;
    const int64_t jlo = max((int64_t)0, r0 - kla), jhi = min(n - 1, r0 + 63 + kua);
    const int64_t span = (jhi - jlo + kResidWaves) / kResidWaves, j1 = min(jhi + 1, jlo + (wave + 1) * span);
    cplx acc = mk(0.0, 0.0);
#pragma unroll 8
    for (int64_t j = jlo + wave * span; j < j1; ++j) {
        const int64_t d = j - i, dc = max((int64_t)-kla, min((int64_t)kua, d));
        const cplx v = A[(kua - dc) + j * lda];
        acc = csel(d == dc, fma_c(acc, v, x[j]), acc);
    }
    // B x, and the entries of u and x for the norms, while the other wavefronts' loads are on their way
    cplx bx = mk(0.0, 0.0), ui = mk(0.0, 0.0), xi = mk(0.0, 0.0);
    if (wave == 0 && i < n) {
        ui = u[i];
        xi = x[i];
        bx = xi;
        if (B != nullptr) {
            const int ldb = klb + kub + 1;
            const int elo = (int)max((int64_t)-klb, -i), ehi = (int)min((int64_t)kub, n - 1 - i);
            bx = mk(0.0, 0.0);
            for (int d = elo; d <= ehi; ++d) bx = fma_c(bx, B[(int64_t)(kub - d) + (i + d) * ldb], x[i + d]);
        }
    }
    if (wave > 0) part[wave - 1][lane] = acc;
    __syncthreads();
    if (wave > 0) return;
    double nr = 0.0, nx = 0.0, nu = 0.0;
    if (i < n) {
#pragma unroll
        for (int w = 0; w < kResidWaves - 1; ++w) acc = acc + part[w][lane];
        acc = fma_c(ui - acc, sigma, bx);
        r[i] = acc;
        nr = cabs(acc);
        nx = cabs(xi);
        nu = cabs(ui);
    }
    nr = wave_max64(nr);
    nx = wave_max64(nx);
    nu = wave_max64(nu);
    if (lane == 0) {
        const unsigned long long o0 = atomic_max_nonneg(norms + 0, nr), o1 = atomic_max_nonneg(norms + 1, nx),
                                 o2 = atomic_max_nonneg(norms + 2, nu);
        if (rs.flags != nullptr) {
            // the norms' atomics have returned before the count goes up (nothing else of this
            // workgroup is read by another before the kernel ends: no fence)
            asm volatile("" ::"v"(o0), "v"(o1), "v"(o2) : "memory");
            if (atomicAdd(norms + 5, 1ull) + 1 == gridDim.x) {
                const double vr = __longlong_as_double((long long)atomicMax(norms + 0, 0ull));
                const double vx = __longlong_as_double((long long)atomicMax(norms + 1, 0ull));
                const double vu = __longlong_as_double((long long)atomicMax(norms + 2, 0ull));
                norms[5] = 0ull;
                refine_check(rs, vr, vx, vu, cnorm, tol, last);
            }
        }
    }
}

// ||A - sigma B||_inf into norms[0] (bit pattern).  Rows and columns are walked as in
// k_band_resid.
__global__ __launch_bounds__(256) void k_band_rownorm(int64_t n, const cplx* __restrict__ A, int kla, int kua,
                                                      const cplx* __restrict__ B, int klb, int kub, cplx sigma,
                                                      unsigned long long* out) {
    __shared__ double part[3][64];
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = r0 + lane;
    const int lda = kla + kua + 1, ldb = klb + kub + 1;
    const int lo = -max(kla, B ? klb : 0), hi = max(kua, B ? kub : 0);
    const int64_t jlo = max((int64_t)0, r0 + lo), jhi = min(n - 1, r0 + 63 + hi);
    const int64_t span = (jhi - jlo + 4) / 4, j1 = min(jhi + 1, jlo + (wave + 1) * span);
    double s = 0.0;
#pragma unroll 4
    for (int64_t j = jlo + wave * span; j < j1; ++j) {
        const int64_t dd = j - i, da = max((int64_t)-kla, min((int64_t)kua, dd));
        const cplx va = A[(kua - da) + j * lda];
        cplx c = csel(dd == da, va, mk(0.0, 0.0));
        if (B != nullptr) {
            const int64_t db = max((int64_t)-klb, min((int64_t)kub, dd));
            const cplx vb = B[(kub - db) + j * ldb];
            c = fms(c, sigma, csel(dd == db, vb, mk(0.0, 0.0)));
        } else if (dd == 0) {
            c = c - sigma;
        }
        s += cabs(c);
    }
    if (wave > 0) part[wave - 1][lane] = s;
    __syncthreads();
    if (wave > 0) return;
    s = (i < n) ? ((s + part[0][lane]) + part[1][lane]) + part[2][lane] : 0.0;
    s = wave_max64(s);
    if (lane == 0) atomic_max_nonneg(out, s);
}

// state[0] = refinement active (starts as *active, or 1), norms cleared
__global__ void k_refine_start(const int* active, RefineState st) {
    st.flags[0] = (active == nullptr || *active != 0) ? 1 : 0;
    st.norms[0] = st.norms[1] = st.norms[2] = 0ull;
}

__global__ __launch_bounds__(256) void k_axpy_gated(int64_t n, cplx* __restrict__ x, const cplx* __restrict__ d,
                                                    const int* gate) {
    if (*gate == 0) return;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) x[i] = x[i] + d[i];
}

simm_status band_inf_norm(int64_t n, const cplx* A, int kla, int kua, const cplx* B, int klb, int kub, cplx sigma,
                          unsigned long long* out, double* host, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(1), 0, st, out, 1);
    hipLaunchKernelGGL(k_band_rownorm, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, st, n, A, kla, kua, B, klb, kub,
                       sigma, out);
    unsigned long long bits = 0;
    SIMM_HIP_TRY(hipMemcpyAsync(&bits, out, sizeof(bits), hipMemcpyDeviceToHost, st));
    SIMM_HIP_TRY(hipStreamSynchronize(st));
    std::memcpy(host, &bits, sizeof(double));
    return SIMM_OK;
}

// u_i = 1 + ((i mod 7) - 3) / 4 + i ((i mod 5) - 2) / 3: a fixed right-hand side with no
// zero entries and no structure aligned with a block partition
__global__ __launch_bounds__(256) void k_probe_rhs(int64_t n, cplx* __restrict__ u) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) u[i] = mk(1.0 + (double)((i % 7) - 3) / 4.0, (double)((i % 5) - 2) / 3.0);
}

simm_status solve_backward_error(const SpikeFactor& f, const RefinePencil& pen, double* eta, hipStream_t st) {
    const int64_t n = f.n;
    const int64_t n16 = (n + 15) / 16 * 16;
    void* mem = nullptr;
    SIMM_HIP_TRY(device_malloc_ordered(&mem, sizeof(cplx) * 3 * (size_t)n16 + 256, st));
    struct Free {
        void* q;
        hipStream_t st;
        ~Free() { device_free_ordered(q, st); }
    } fr{mem, st};
    cplx* u = reinterpret_cast<cplx*>(mem);
    cplx* x = u + n16;
    cplx* r = x + n16;
    unsigned long long* norms = reinterpret_cast<unsigned long long*>(r + n16);
    int* gate = reinterpret_cast<int*>(norms + 4);
    const unsigned blocks = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_probe_rhs, dim3(blocks), dim3(256), 0, st, n, u);
    hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(64), 0, st, norms, 4);
    const int one = 1;
    SIMM_HIP_TRY(hipMemcpyAsync(gate, &one, sizeof(int), hipMemcpyHostToDevice, st));
    ChainSlots slots;   // released (after a synchronize) when this returns
    SIMM_TRY(slots.acquire(spike_chain_weight(f), st));
    SIMM_TRY(spike_apply(f, u, x, nullptr, st));
    hipLaunchKernelGGL(k_band_resid, dim3((unsigned)((n + 63) / 64)), dim3(64 * kResidWaves), 0, st, n, pen.A, pen.kla, pen.kua,
                       pen.B, pen.klb, pen.kub, pen.sigma, (const cplx*)u, (const cplx*)x, r, norms, (const int*)gate,
                       RefineState{}, 0.0, 0.0, 0);
    SIMM_HIP_TRY(hipGetLastError());
    unsigned long long nb[3] = {0, 0, 0};
    SIMM_HIP_TRY(hipMemcpyAsync(nb, norms, sizeof(nb), hipMemcpyDeviceToHost, st));
    SIMM_HIP_TRY(hipStreamSynchronize(st));
    double v[3];
    std::memcpy(v, nb, sizeof(v));
    const double den = pen.cnorm * v[1] + v[2];
    *eta = den > 0.0 ? v[0] / den : 0.0;
    if (!std::isfinite(v[0]) || !std::isfinite(v[1])) *eta = INFINITY;
    return SIMM_OK;
}

simm_status refine_apply(const SpikeFactor& f, const RefinePencil& pen, const RefineState& rs, const cplx* u, cplx* y,
                         const int* active, hipStream_t st) {
    const int64_t n = f.n;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    const int* gate = rs.flags;
    hipLaunchKernelGGL(k_refine_start, dim3(1), dim3(1), 0, st, active, rs);
    SIMM_TRY(spike_apply(f, u, y, active, st));
    for (int k = 0; k <= kRefineMaxSteps; ++k) {
        hipLaunchKernelGGL(k_band_resid, dim3((unsigned)((n + 63) / 64)), dim3(64 * kResidWaves), 0, st, n, pen.A, pen.kla,
                           pen.kua, pen.B, pen.klb, pen.kub, pen.sigma, u, (const cplx*)y, rs.r, rs.norms, gate, rs,
                           pen.cnorm, kRefineTol, k == kRefineMaxSteps ? 1 : 0);
        if (k == kRefineMaxSteps) break;
        SIMM_TRY(spike_apply(f, rs.r, rs.d, gate, st));
        hipLaunchKernelGGL(k_axpy_gated, dim3(blocks), dim3(256), 0, st, n, y, (const cplx*)rs.d, gate);
    }
    SIMM_HIP_TRY(hipGetLastError());
    return SIMM_OK;
}

}  // namespace simm
