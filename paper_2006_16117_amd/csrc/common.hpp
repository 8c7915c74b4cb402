// Shared device/host helpers of the SIM-M HIP library (gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <string>

#include "simm.h"

namespace simm {

// ---------------------------------------------------------------------------
// complex<double> as two interleaved doubles
// ---------------------------------------------------------------------------
struct cplx {
    double re, im;
};

__host__ __device__ inline cplx mk(double r, double i) { return cplx{r, i}; }
__host__ __device__ inline cplx operator+(cplx a, cplx b) { return cplx{a.re + b.re, a.im + b.im}; }
__host__ __device__ inline cplx operator-(cplx a, cplx b) { return cplx{a.re - b.re, a.im - b.im}; }
__host__ __device__ inline cplx operator-(cplx a) { return cplx{-a.re, -a.im}; }
__host__ __device__ inline cplx operator*(cplx a, cplx b) {
    return cplx{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__host__ __device__ inline cplx operator*(double s, cplx a) { return cplx{s * a.re, s * a.im}; }
__host__ __device__ inline cplx conj(cplx a) { return cplx{a.re, -a.im}; }
__host__ __device__ inline double norm2(cplx a) { return a.re * a.re + a.im * a.im; }
__host__ __device__ inline double cabs1(cplx a) { return fabs(a.re) + fabs(a.im); }
__host__ __device__ inline double cabs(cplx a) { return hypot(a.re, a.im); }
// a - b * c  (fused form used in the sweeps and eliminations)
__host__ __device__ inline cplx fms(cplx a, cplx b, cplx c) {
    return cplx{a.re - b.re * c.re + b.im * c.im, a.im - b.re * c.im - b.im * c.re};
}
// a + b * c
__host__ __device__ inline cplx fma_c(cplx a, cplx b, cplx c) {
    return cplx{a.re + b.re * c.re - b.im * c.im, a.im + b.re * c.im + b.im * c.re};
}
// a + conj(b) * c
__host__ __device__ inline cplx fma_cj(cplx a, cplx b, cplx c) {
    return cplx{a.re + b.re * c.re + b.im * c.im, a.im + b.re * c.im - b.im * c.re};
}
// c ? a : b, component-wise (a struct-valued ?: can be lowered through scratch memory)
__host__ __device__ inline cplx csel(bool c, cplx a, cplx b) { return cplx{c ? a.re : b.re, c ? a.im : b.im}; }

// complex<float>: the storage and arithmetic of the FP32 band factor (same operations)
struct cplxf {
    float re, im;
};
__host__ __device__ inline cplxf operator+(cplxf a, cplxf b) { return cplxf{a.re + b.re, a.im + b.im}; }
__host__ __device__ inline cplxf operator-(cplxf a, cplxf b) { return cplxf{a.re - b.re, a.im - b.im}; }
__host__ __device__ inline cplxf operator*(cplxf a, cplxf b) {
    return cplxf{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__host__ __device__ inline float cabs1(cplxf a) { return fabsf(a.re) + fabsf(a.im); }
__host__ __device__ inline cplxf fms(cplxf a, cplxf b, cplxf c) {
    return cplxf{a.re - b.re * c.re + b.im * c.im, a.im - b.re * c.im - b.im * c.re};
}
__host__ __device__ inline cplxf csel(bool c, cplxf a, cplxf b) { return cplxf{c ? a.re : b.re, c ? a.im : b.im}; }
// widening / rounding between the two
__host__ __device__ inline cplx widen(cplx a) { return a; }
__host__ __device__ inline cplx widen(cplxf a) { return cplx{(double)a.re, (double)a.im}; }
template <typename C>
__host__ __device__ inline C narrow(cplx a);
template <>
__host__ __device__ inline cplx narrow<cplx>(cplx a) { return a; }
template <>
__host__ __device__ inline cplxf narrow<cplxf>(cplx a) { return cplxf{(float)a.re, (float)a.im}; }
// a / b, scaled to avoid overflow (Smith's method)
__host__ __device__ inline cplx cdiv(cplx a, cplx b) {
    if (fabs(b.re) >= fabs(b.im)) {
        double r = b.im / b.re, d = b.re + b.im * r;
        return cplx{(a.re + a.im * r) / d, (a.im - a.re * r) / d};
    } else {
        double r = b.re / b.im, d = b.im + b.re * r;
        return cplx{(a.re * r + a.im) / d, (a.im * r - a.re) / d};
    }
}

// ---------------------------------------------------------------------------
// Workgroup barrier for LDS traffic only: waits for this wave's LDS operations
// and meets the other waves, without waiting on outstanding global loads (a
// plain __syncthreads() also drains every global load in flight, which defeats
// register prefetching in latency-bound loops).  The "memory" clobber keeps the
// compiler from moving memory accesses across it.
// ---------------------------------------------------------------------------
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// 16-byte (FP64) or 8-byte (FP32) LDS accesses of whole complex entries; every LDS
// buffer is aligned to its entry size.
__device__ inline cplx ldsr(const cplx* p) {
    const double2 v = *reinterpret_cast<const double2*>(p);
    return cplx{v.x, v.y};
}
__device__ inline void ldsw(cplx* p, cplx v) { *reinterpret_cast<double2*>(p) = double2{v.re, v.im}; }
__device__ inline cplxf ldsr(const cplxf* p) {
    const float2 v = *reinterpret_cast<const float2*>(p);
    return cplxf{v.x, v.y};
}
__device__ inline void ldsw(cplxf* p, cplxf v) { *reinterpret_cast<float2*>(p) = float2{v.re, v.im}; }

// ---------------------------------------------------------------------------
// lane exchange within a wavefront (device code)
// ---------------------------------------------------------------------------
template <int CTRL, int ROW_MASK = 0xf>
__device__ inline double dpp_d(double v) {
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(v), __double2loint(v), CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(v), __double2hiint(v), CTRL, ROW_MASK, 0xf, false);
    return __hiloint2double(hi, lo);
}
template <int CTRL, int ROW_MASK = 0xf>
__device__ inline float dpp_d(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}

__device__ inline double rdlane_d(double v, int l) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}
__device__ inline float rdlane_d(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }
__device__ inline cplx rdlane(cplx v, int l) { return cplx{rdlane_d(v.re, l), rdlane_d(v.im, l)}; }
__device__ inline cplxf rdlane(cplxf v, int l) { return cplxf{rdlane_d(v.re, l), rdlane_d(v.im, l)}; }

// Maximum over the wavefront, returned to every lane: DPP within 16-lane rows
// (quad xor 1, quad xor 2, half-row mirror, row mirror), then row broadcasts of
// lanes 15 and 31 carry the row maxima to lane 63.
template <typename R>
__device__ inline R wave_max(R v) {
    v = fmax(v, dpp_d<0xB1>(v));
    v = fmax(v, dpp_d<0x4E>(v));
    v = fmax(v, dpp_d<0x141>(v));
    v = fmax(v, dpp_d<0x140>(v));
    v = fmax(v, dpp_d<0x142, 0xA>(v));
    v = fmax(v, dpp_d<0x143, 0xC>(v));
    return rdlane_d(v, 63);
}

// 1 / u by Smith's scaling (no overflow for any finite nonzero u), without branches.
__device__ inline cplx crecip(cplx u) {
    const bool big = fabs(u.re) >= fabs(u.im);
    const double p = big ? u.re : u.im, q = big ? u.im : u.re;
    const double s = q / p, d = 1.0 / (p + q * s);
    return big ? cplx{d, -s * d} : cplx{s * d, -d};
}
__device__ inline cplxf crecip(cplxf u) {
    const bool big = fabsf(u.re) >= fabsf(u.im);
    const float p = big ? u.re : u.im, q = big ? u.im : u.re;
    const float s = q / p, d = 1.0f / (p + q * s);
    return big ? cplxf{d, -s * d} : cplxf{s * d, -d};
}

// ---------------------------------------------------------------------------
// error reporting (thread-local message behind simm_last_error)
// ---------------------------------------------------------------------------
void set_error(const std::string& msg);
void clear_error();

#define SIMM_HIP_TRY(expr)                                                                  \
    do {                                                                                    \
        hipError_t _e = (expr);                                                             \
        if (_e != hipSuccess) {                                                             \
            ::simm::set_error(std::string(#expr) + ": " + hipGetErrorString(_e));           \
            return (_e == hipErrorOutOfMemory) ? SIMM_ENOMEM : SIMM_EHIP;                   \
        }                                                                                   \
    } while (0)

// internal status of work given up on purpose (a factor computed ahead that is no
// longer needed); never returned through the C ABI
constexpr simm_status SIMM_ECANCELED = static_cast<simm_status>(7);

#define SIMM_TRY(expr)                         \
    do {                                       \
        simm_status _s = (expr);               \
        if (_s != SIMM_OK) return _s;          \
    } while (0)

}  // namespace simm
