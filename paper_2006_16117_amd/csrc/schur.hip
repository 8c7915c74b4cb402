// Schur form H_m = Q T Q^H of the Arnoldi Hessenberg matrix, once per shift.
//
// The shifted Galerkin systems (I + (sigma - z_j) H_m) y_j = beta e_1 of Sec. 2,
// eq. (many), become (I + (sigma - z_j) T) yhat_j = beta Q^H e_1 with y_j = Q yhat_j:
// an upper triangular solve per quadrature point.  Sec. 3.2 of the paper uses an
// eigendecomposition H_m = P D P^{-1} instead; the unitary Schur basis gives the same
// rational functions of z without inverting a possibly ill-conditioned P.  The
// diagonal of T holds the eigenvalues theta of H_m (Ritz values sigma + 1/theta).
//
// Method: complex single-shift QR iteration on the Hessenberg matrix (Wilkinson
// shift from the trailing 2x2 block, exceptional shifts after 10 and 20 stalled
// iterations, deflation when |h_{k,k-1}| <= eps (|h_{k-1,k-1}| + |h_{k,k}|)), each
// sweep in two phases, H - mu I = Q_s R by Givens rotations from the left over the whole
// rows, then R Q_s + mu I and Q Q_s by the same rotations from the right, so that the
// full upper triangular T results.
//
// A sweep is a serial chain of rotations (about 9,400 for m = 80 in all), so what counts
// is the latency of one, not arithmetic:
//  * left phase, one wavefront, a lane per column: the row that the next rotation
//    works on stays in registers, so a rotation's chain is a lane read of its leading
//    entry, one reciprocal square root and a few multiply-adds, with no trip through LDS.
//    (The rotation is the unitary [conj x, conj y; -y, x] / n, n^2 = |x|^2 + |y|^2: one
//    reciprocal square root, where a real cosine takes two square roots and two
//    divisions; the products are formed beside the root and scaled by 1 / n at the end.)
//  * right phase, a lane per row of H or Q, on other wavefronts: rotation k may be
//    applied from the right once the left phase is past rotation k + 1 (the rows it meets
//    are then final), so these wavefronts follow the left phase two rotations behind, by a
//    progress count in LDS, and a sweep takes little more than its left phase.
// The kernel: m = 40 0.76 ms, m = 80 3.4 ms, m = 120 7.2 to 7.5 ms; 2.3, 8.5 and 18.9 ms (with
// the call) when every rotation went through LDS twice on one wavefront and a second kernel
// replayed the rotations on Q.  0.29 to 0.36 us a rotation: 75 instructions of the left phase,
// most of them FP64 and each waiting for the one before.
#include "common.hpp"
#include "kernels.hpp"

namespace simm {

namespace {

__device__ inline int hoff(int j) { return j * (j + 5) / 2; }   // column j holds rows 0 .. j+2

__device__ inline cplx csqrt_d(cplx z) {
    // principal square root (z is of the size of H_m's entries squared: its own squares may leave
    // the range that those of the entries stay in)
    const double r = hypot(z.re, z.im);
    if (r == 0.0) return mk(0.0, 0.0);
    const double a = sqrt(0.5 * (r + fabs(z.re)));
    const double b = z.im / (2.0 * a);
    if (z.re >= 0.0) return mk(a, b);
    return (z.im >= 0.0) ? mk(fabs(b), a) : mk(fabs(b), -a);
}

// 1 / sqrt(a), a > 0: the hardware's estimate (about 2^-25) and one third-order step
__device__ inline double rsqrt_d(double a) {
    const double y = __builtin_amdgcn_rsq(a);
    const double e = fma(-a * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

constexpr int MAX_SCHUR_M = 128;
constexpr size_t SCHUR_LDS = 160 * 1024;

// What the first wavefront tells the others about a sweep.
struct SweepInfo {
    cplx mu;
    int l, ihi, stop;
    int prog;   // rotations of the sweep done so far, as their index + 1 (left_phase)
};

// Largest k <= ihi with a negligible subdiagonal entry H(k, k-1) (0 if none), by one
// wavefront, every lane testing its own k (lane + 1, lane + 65).
__device__ inline int deflation_point(const cplx* Hs, int ihi, int lane) {
    const double eps = 2.220446049250313e-16;
    auto H = [&](int i, int j) -> cplx { return Hs[hoff(j) + i]; };
    double dsum = -1.0;   // sum of |diag| over 0..ihi, only if some test needs it
    int l = 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int k = lane + 1 + 64 * u;
        bool small = false;
        double tst = 0.0;
        if (k <= ihi) {
            tst = cabs1(H(k - 1, k - 1)) + cabs1(H(k, k));
            small = tst != 0.0 && cabs1(H(k, k - 1)) <= eps * tst;
        }
        if (__ballot(k <= ihi && tst == 0.0)) {
            if (dsum < 0.0) {
                double acc = 0.0;
                for (int i = lane; i <= ihi; i += 64) acc += cabs1(H(i, i));
#pragma unroll
                for (int msk = 32; msk >= 1; msk >>= 1) acc += __shfl_xor(acc, msk, 64);
                dsum = (acc == 0.0) ? 1.0 : acc;
            }
            if (k <= ihi && tst == 0.0) small = cabs1(H(k, k - 1)) <= eps * dsum;
        }
        const unsigned long long bal = __ballot(small);
        if (bal) l = 64 * u + 64 - __clzll((long long)bal);
    }
    return l;
}

// The progress count: relaxed accesses (a wavefront's LDS accesses execute in order; the
// compiler keeps them in order at the empty asm)
__device__ inline void set_progress(int* p, int v) {
    asm volatile("" ::: "memory");
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline int get_progress(int* p) {
    const int v = __builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    asm volatile("" ::: "memory");
    return v;
}

// Left phase of a sweep, by one wavefront: rows l .. ihi of H - mu I times the rotations,
// lane j holding columns j + 64 u (u < W); rot[2k], rot[2k+1] = x / n, y / n; *prog = k + 1
// after rotation k.  LDS accesses of a wavefront execute in order, so a reader that sees
// prog = k + 1 sees the rows up to k and the rotations before it.  No branch in the loop:
// lanes with nothing to write write `trash`, so that the wait for the row read ahead does
// not include the writes.
template <int W>
__device__ __forceinline__ void left_phase(cplx* Hs, int m, int l, int ihi, cplx mu, cplx* rot, int* prog,
                                           cplx* trash, int lane) {
    cplx cur[W], h[W];
    int col[W], off[W];
    // row r of this lane's column u; rows below the stored ones read the last stored entry
    // (not used: column j takes part in the rotations of rows up to j only)
    auto row = [&](int u, int r) {
        const cplx v = ldsr(Hs + off[u] + min(r, col[u] + 2));
        return csel(r == col[u], v - mu, v);
    };
#pragma unroll
    for (int u = 0; u < W; ++u) {
        col[u] = min(lane + 64 * u, m - 1);
        off[u] = hoff(col[u]);
        cur[u] = row(u, l);
        h[u] = row(u, l + 1);
    }
    for (int k = l; k < ihi; ++k) {
        cplx raw[W];
        const int rn = min(k + 2, ihi);
#pragma unroll
        for (int u = 0; u < W; ++u) raw[u] = ldsr(Hs + off[u] + min(rn, col[u] + 2));
        cplx x, y;
        if (W == 1 || k < 64) {
            x = rdlane(cur[0], k & 63);
            y = rdlane(h[0], k & 63);
        } else {
            x = rdlane(cur[W - 1], k & 63);
            y = rdlane(h[W - 1], k & 63);
        }
        const double n2 = (x.re * x.re + x.im * x.im) + (y.re * y.re + y.im * y.im);
        const bool none = !(n2 > 0.0);      // nothing to rotate: the identity
        x.re = none ? 1.0 : x.re;
        const double rn2 = rsqrt_d(none ? 1.0 : n2);
        cplx nw[W];
#pragma unroll
        for (int u = 0; u < W; ++u) {
            // new row k: (conj(x) cur + conj(y) h) / n; row k + 1 carried on: (x h - y cur) / n
            const cplx a = fma_cj(mk(x.re * cur[u].re + x.im * cur[u].im, x.re * cur[u].im - x.im * cur[u].re), y, h[u]);
            const cplx b = fms(x * h[u], y, cur[u]);
            nw[u] = mk(a.re * rn2, a.im * rn2);
            cur[u] = mk(b.re * rn2, b.im * rn2);
        }
#pragma unroll
        for (int u = 0; u < W; ++u) {
            const int j = lane + 64 * u;
            ldsw((j >= k && j < m) ? Hs + off[u] + k : trash, nw[u]);
        }
        const cplx xr = mk(x.re * rn2, x.im * rn2), yr = mk(y.re * rn2, y.im * rn2);
        ldsw(lane < 2 ? rot + 2 * k + lane : trash, csel(lane == 0, xr, yr));
        set_progress(prog, k + 1);
#pragma unroll
        for (int u = 0; u < W; ++u) h[u] = csel(rn == col[u], raw[u] - mu, raw[u]);
    }
#pragma unroll
    for (int u = 0; u < W; ++u) {
        const int j = lane + 64 * u;
        ldsw((j >= ihi && j < m) ? Hs + off[u] + ihi : trash, cur[u]);
    }
    set_progress(prog, ihi + 2);
}

// Right phase on one row, behind the left phase: columns l .. ihi times the rotations'
// conjugate transposes.  get(k) reads the row's entry of column k (once the left phase is
// past the rows that meet it), put(k, v) writes it; PF columns are read ahead (one from
// LDS, several from global memory, whose loads take longer than a rotation; rows of Q only,
// which do not wait for the left phase but for its rotations).
template <int PF, typename Get, typename Put>
__device__ __forceinline__ void right_phase(int l, int ihi, const cplx* rot, int* prog, Get get, Put put) {
    int ready = 0;
    auto wait = [&](int need) {   // until *prog >= need (every sweep ends at ihi + 2)
        while (ready < need) ready = get_progress(prog);
    };
    wait(l + 2);
    cplx cur = get(l), h[PF];
#pragma unroll
    for (int s = 0; s < PF; ++s) h[s] = get(min(l + 1 + s, ihi));
    for (int k0 = l; k0 < ihi; k0 += PF) {
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            const int k = k0 + s;
            if (PF > 1 && k >= ihi) break;
            // column k + 2 (PF = 1) is final in the rows up to k + 2 after rotation k + 2.
            // What the step reads is read behind the count, in one trip to LDS: valid if the
            // count has come far enough, else read again.
            const int need = min(k + 3, ihi + 2), kn = min(k + 1 + PF, ihi);
            cplx xr, yr, hn;
            while (true) {
                int p = ready;
                if (ready < need) p = __hip_atomic_load(prog, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                asm volatile("" ::: "memory");
                xr = ldsr(rot + 2 * k);
                yr = ldsr(rot + 2 * k + 1);
                hn = get(kn);
                asm volatile("" ::: "memory");
                ready = __builtin_amdgcn_readfirstlane(p);
                if (ready >= need) break;
            }
            // (c_k, c_{k+1}) G^H: c_k' = cur xr + h yr; carried on: h conj(xr) - cur conj(yr)
            put(k, fma_c(cur * xr, h[s], yr));
            cur = fms(h[s] * conj(xr), cur, conj(yr));
            h[s] = hn;
        }
    }
    put(ihi, cur);
}

}  // namespace

// One workgroup of 2 W + 1 wavefronts (W = 1 up to m = 64): wavefront 0 tests for
// deflation, picks the shift and does the left phase; wavefronts 1 .. W take the rows of H
// and the last W the rows of Q.  H packed by columns in LDS, Q in LDS where both fit
// (QLDS, m <= 80), else in global memory (each lane works on a row of its own, its next
// columns' loads in flight).
template <int W, bool QLDS>
__global__ __launch_bounds__(64 * (2 * W + 1)) void k_hess_schur(const cplx* __restrict__ Hin, int ldh, int m,
                                                                 double beta, cplx* T_out, cplx* Q, cplx* g,
                                                                 cplx* qlast, int* status) {
    constexpr int NW = 2 * W + 1;
    extern __shared__ double2 schur_sm[];
    cplx* Hs = reinterpret_cast<cplx*>(schur_sm);
    cplx* rot = Hs + hoff(m);
    cplx* trash = rot + 2 * m;   // one entry a lane
    SweepInfo* info = reinterpret_cast<SweepInfo*>(trash + 64);
    cplx* Qs = QLDS ? reinterpret_cast<cplx*>(info + 1) : Q;
    int* prog = &info->prog;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the m x m Hessenberg part (rows 0 .. j+1 of column j; the slot below stays zero)
    for (int j = wave; j < m; j += NW)
        for (int i = lane; i <= j + 2; i += 64)
            Hs[hoff(j) + i] = (i <= j + 1 && i < m) ? Hin[i + (int64_t)j * ldh] : mk(0.0, 0.0);
    const int row = lane + 64 * (wave - W - 1);   // of Q, for the last W wavefronts
    if (wave > W && row < m)
        for (int k = 0; k < m; ++k) ldsw(Qs + k * m + row, mk((k == row) ? 1.0 : 0.0, 0.0));
    __syncthreads();

    int ihi = m - 1, its = 0;   // wavefront 0's
    while (true) {
        cplx mu = mk(0.0, 0.0);
        if (wave == 0) {
            auto H = [&](int i, int j) -> cplx { return Hs[hoff(j) + i]; };
            int l = 0, stop = 0;
            while (ihi > 0) {
                l = deflation_point(Hs, ihi, lane);
                if (l > 0 && lane == 0) Hs[hoff(l - 1) + l] = mk(0.0, 0.0);
                if (l < ihi) break;
                --ihi;
                its = 0;
            }
            if (ihi <= 0) {
                stop = 1;
            } else if (its >= 40) {
                stop = 2;
            } else {
                ++its;
                if (its == 10) {
                    const cplx d = H(ihi, ihi);
                    mu = mk(d.re + 0.75 * fabs(H(ihi, ihi - 1).re), d.im);
                } else if (its == 20) {
                    const cplx d = H(l, l);
                    mu = mk(d.re + 0.75 * fabs(H(l + 1, l).re), d.im);
                } else {
                    const cplx a = H(ihi - 1, ihi - 1), b = H(ihi - 1, ihi), c = H(ihi, ihi - 1), d = H(ihi, ihi);
                    const cplx half = mk(0.5 * (a.re - d.re), 0.5 * (a.im - d.im));
                    const cplx disc = csqrt_d(half * half + b * c);
                    const cplx tr2 = mk(0.5 * (a.re + d.re), 0.5 * (a.im + d.im));
                    const cplx m1 = tr2 + disc, m2 = tr2 - disc;
                    mu = (norm2(m1 - d) <= norm2(m2 - d)) ? m1 : m2;
                }
            }
            if (lane == 0) {
                info->mu = mu;
                info->l = l;
                info->ihi = ihi;
                info->stop = stop;
                set_progress(prog, 0);
            }
        }
        __syncthreads();
        const int stop = info->stop, l = info->l, hi = info->ihi;
        if (stop) {
            if (tid == 0) *status = stop - 1;
            break;
        }
        if (wave == 0) {
            left_phase<W>(Hs, m, l, hi, mu, rot, prog, trash + lane, lane);
        } else if (wave <= W) {
            const int i = lane + 64 * (wave - 1);
            mu = info->mu;
            if (i <= hi)
                right_phase<1>(l, hi, rot, prog,
                               [&](int k) { return csel(i <= k, ldsr(Hs + hoff(k) + min(i, k)), mk(0.0, 0.0)); },
                               [&](int k, cplx v) {
                                   ldsw(i <= k + 1 ? Hs + hoff(k) + i : trash + lane, csel(i == k, v + mu, v));
                               });
        } else if (row < m) {
            right_phase<QLDS ? 1 : 8>(l, hi, rot, prog, [&](int k) { return ldsr(Qs + k * m + row); },
                                      [&](int k, cplx v) { ldsw(Qs + k * m + row, v); });
        }
        __syncthreads();
    }
    __syncthreads();
    // packed upper triangle; Q with the rows that the solves need
    for (int j = wave; j < m; j += NW)
        for (int i = lane; i <= j; i += 64) T_out[j * (j + 1) / 2 + i] = Hs[hoff(j) + i];
    if (wave > W && row < m) {
        if (QLDS)
            for (int k = 0; k < m; ++k) Q[k * m + row] = Qs[k * m + row];
        if (row == 0)
            for (int k = 0; k < m; ++k) {
                const cplx q = Qs[k * m];
                g[k] = mk(beta * q.re, -beta * q.im);
            }
        if (row == m - 1)
            for (int k = 0; k < m; ++k) qlast[k] = Qs[k * m + row];
    }
}

simm_status hess_schur(const cplx* H, int ldh, int m, double beta, SchurOut out, int* status, hipStream_t st) {
    if (m < 1 || m > MAX_SCHUR_M) {
        set_error("Krylov dimension outside 1..128");
        return SIMM_EUNSUPPORTED;
    }
    const size_t base = sizeof(cplx) * (size_t)(m * (m + 5) / 2 + 2 * m + 64) + sizeof(SweepInfo);
    const size_t q = sizeof(cplx) * (size_t)m * m;
    const bool qlds = base + q <= SCHUR_LDS;
    const size_t lds = base + (qlds ? q : 0);
    if (m <= 64)
        hipLaunchKernelGGL((k_hess_schur<1, true>), dim3(1), dim3(192), lds, st, H, ldh, m, beta, out.T, out.Q, out.g,
                           out.qlast, status);
    else if (qlds)
        hipLaunchKernelGGL((k_hess_schur<2, true>), dim3(1), dim3(320), lds, st, H, ldh, m, beta, out.T, out.Q, out.g,
                           out.qlast, status);
    else
        hipLaunchKernelGGL((k_hess_schur<2, false>), dim3(1), dim3(320), lds, st, H, ldh, m, beta, out.T, out.Q, out.g,
                           out.qlast, status);
    SIMM_HIP_TRY(hipGetLastError());
    return SIMM_OK;
}

}  // namespace simm
