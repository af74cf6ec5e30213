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
enum { GANG_NONE = 0, GANG_GO = 1, GANG_LEFT = 2, GANG_FAILED = 3, GANG_FEW = 4 };

// The words of a matrix's state.  The gang's form in registers has the first two,
// its form in memory the next two, at the same places from its own pointer on.
enum {
    GS_STATE = 0,     // GANG_...
    GS_ARRIVED = 1,   // workgroups that have counted in
    GS_MEM = 2,       // where the form in memory has its two
    GS_CHIP = 4,      // the whole chip is this gang's (until trd_single_kernel gives it back)
    GS_SKIP = 5,      // whole-chip gangs to come that leave at once
    GS_SKIP_NEXT = 6, // how many did so after the last one that could not gather
    GS_TRIED = 7      // the last whole-chip gang waited for its workgroups
};

// A workgroup of a form in registers counts in and waits for all P of them: GANG_GO, or
// GANG_LEFT when they have not come in time.
__device__ inline int gather(int* state, int P, long long gate, int* chip) {
    const long long t0 = wall_clock64();
    if (atomicAdd(&state[GS_ARRIVED], 1) == P - 1 && atomicCAS(&state[GS_STATE], GANG_NONE, GANG_GO) == GANG_NONE &&
        state[GS_CHIP])
        atomicExch(chip, 2);
    int st;
    while ((st = __hip_atomic_load(&state[GS_STATE], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == GANG_NONE) {
        if (wall_clock64() - t0 >= gate) atomicCAS(&state[GS_STATE], GANG_NONE, GANG_LEFT);
    }
    return st;
}
// A workgroup of a form in memory counts in and waits for the others.  Returns its
// number; P is how many they are, 0 where it takes no part.  `full` of them where
// these arrive within the time that a whole-chip gang has, else the `few` that fit
// the chip beside anything (a quarter of it).
__device__ inline int gather_in_memory(int* state, int full, int few, long long gate, int& P) {
    const long long t0 = wall_clock64();
    const int b = atomicAdd(&state[GS_ARRIVED], 1);
    P = 0;
    if (b >= full) return b;
    if (b == full - 1) atomicCAS(&state[GS_STATE], GANG_NONE, GANG_GO);
    int st;
    while ((st = __hip_atomic_load(&state[GS_STATE], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == GANG_NONE) {
        const long long w = wall_clock64() - t0;
        if (w >= gate)
            atomicCAS(&state[GS_STATE], GANG_NONE, GANG_LEFT);
        else if (w >= CHIP_GATE_MS * TICKS &&
                 __hip_atomic_load(&state[GS_ARRIVED], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= few)
            atomicCAS(&state[GS_STATE], GANG_NONE, GANG_FEW);
    }
    P = st == GANG_GO ? full : st == GANG_FEW ? few : 0;
    return b;
}

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

// acc += a b, a fused multiply-add per real product
__device__ __forceinline__ void fma_(double& acc, double a, double b) { acc = fma(a, b, acc); }
__device__ __forceinline__ void fma_(cplx& acc, cplx a, cplx b) {
    acc.x = fma(-a.y, b.y, fma(a.x, b.x, acc.x));
    acc.y = fma(a.y, b.x, fma(a.x, b.y, acc.y));
}


// H_k = I - tau v v^H from alpha = x_{k+1} and |x_{k+2..}|^2 (as in ks_hetrd.hip).
template <typename T>
__device__ __forceinline__ void form_reflector(T alpha, double xn2, T& sc, T& tv, double& beta) {
    const double ar = re_(alpha), ai = im_(alpha);
    if (xn2 == 0.0 && ai == 0.0) {
        tv = zero_<T>();
        beta = ar;
        sc = zero_<T>();
    } else {
        beta = -copysign(sqrt(fma(ar, ar, fma(ai, ai, xn2))), ar);
        tv = mk_<T>((beta - ar) / beta, -ai / beta);
        sc = inv_(alpha - from_re<T>(beta));
    }
}

__device__ __forceinline__ double mul_(double a, double b) { return a * b; }
__device__ __forceinline__ cplx mul_(cplx a, cplx b) {
    return mk(fma(-a.y, b.y, a.x * b.x), fma(a.y, b.x, a.x * b.y));
}
// acc += s a, |a|^2, Re(conj(a) b)
__device__ __forceinline__ void add_scaled(double& acc, double s, double a) { acc = fma(s, a, acc); }
__device__ __forceinline__ void add_scaled(cplx& acc, double s, cplx a) { acc = mk(fma(s, a.x, acc.x), fma(s, a.y, acc.y)); }
__device__ __forceinline__ void add_dot(double& acc, double a, double b) { acc = fma(a, b, acc); }
__device__ __forceinline__ void add_dot(double& acc, cplx a, cplx b) { acc = fma(a.y, b.y, fma(a.x, b.x, acc)); }
template <typename T>
__device__ __forceinline__ void add_abs2(double& acc, T a) {
    add_dot(acc, a, a);
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
