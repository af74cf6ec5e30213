// ks_gang.hpp -- what the gangs of workgroups of the tridiagonalisation share: the
// exchange whose data are their own flags, the gate, and the reflector.
#pragma once

#include "ks_internal.hpp"

namespace ks {

namespace {

typedef unsigned long long u64;
constexpr u64 EMPTY = 0x7ff4a5a5deadbeefULL;  // a signalling NaN: no operation returns it
constexpr long long TICKS = 100000;           // wall_clock64() ticks per millisecond
constexpr long long GATE_MS = 1000, CHIP_GATE_MS = 3, WAIT_MS = 4000;
enum { GANG_NONE = 0, GANG_GO = 1, GANG_LEFT = 2, GANG_FAILED = 3 };

__device__ __forceinline__ void publish(double* p, double v) {
    u64 b = (u64)__double_as_longlong(v);
    if (b == EMPTY) b ^= 1;
    __hip_atomic_store((u64*)p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish(cplx* p, cplx v) {
    publish(&p->x, v.x);
    publish(&p->y, v.y);
}
__device__ __forceinline__ void empty_out(double* p) {
    __hip_atomic_store((u64*)p, EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void empty_out(cplx* p) {
    empty_out(&p->x);
    empty_out(&p->y);
}
__device__ __forceinline__ double peek(const double* p) {
    return __longlong_as_double((long long)__hip_atomic_load((const u64*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ cplx peek(const cplx* p) { return mk(peek(&p->x), peek(&p->y)); }
__device__ __forceinline__ bool is_empty(double v) { return (u64)__double_as_longlong(v) == EMPTY; }
template <typename T>
__device__ __forceinline__ T empty_();
template <>
__device__ __forceinline__ double empty_<double>() { return __longlong_as_double((long long)EMPTY); }
template <>
__device__ __forceinline__ cplx empty_<cplx>() { return mk(empty_<double>(), empty_<double>()); }
__device__ __forceinline__ bool is_empty(cplx v) { return is_empty(v.x) || is_empty(v.y); }

template <typename T>
__device__ __forceinline__ T mk_(double re, double im);
template <>
__device__ __forceinline__ double mk_<double>(double re, double) { return re; }
template <>
__device__ __forceinline__ cplx mk_<cplx>(double re, double im) { return mk(re, im); }

// H_k = I - tau v v^H from alpha = x_{k+1} and |x_{k+2..}|^2 (as in ks_hetrd.hip).
template <typename T>
__device__ __forceinline__ void form_reflector(T alpha, double xn2, T& sc, T& tv, double& beta) {
    const double ar = re_(alpha), ai = im_(alpha);
    if (xn2 == 0.0 && ai == 0.0) {
        tv = zero_<T>();
        beta = ar;
        sc = zero_<T>();
    } else {
        beta = -copysign(sqrt(ar * ar + ai * ai + xn2), ar);
        tv = mk_<T>((beta - ar) / beta, -ai / beta);
        sc = inv_(alpha - from_re<T>(beta));
    }
}

// acc += a b, a fused multiply-add per real product
__device__ __forceinline__ void fma_(double& acc, double a, double b) { acc = fma(a, b, acc); }
__device__ __forceinline__ void fma_(cplx& acc, cplx a, cplx b) {
    acc.x = fma(-a.y, b.y, fma(a.x, b.x, acc.x));
    acc.y = fma(a.y, b.x, fma(a.x, b.y, acc.y));
}

// a += v u + p w.  The products are added up before they meet a, which is then
// rounded once: rounded at every product, the entries of a matrix that stays in
// registers through all its columns had twice (complex) and 1.5 times (real) the
// error of one that takes 32 columns at a time.
__device__ __forceinline__ void rank2_(double& a, double v, double u, double p, double w) { a += fma(p, w, v * u); }
__device__ __forceinline__ void rank2_(cplx& a, cplx v, cplx u, cplx p, cplx w) {
    cplx d = mk(v.x * u.x, v.x * u.y);
    d.x = fma(-v.y, u.y, d.x);
    d.y = fma(v.y, u.x, d.y);
    fma_(d, p, w);
    a = mk(a.x + d.x, a.y + d.y);
}

}  // namespace

}  // namespace ks
