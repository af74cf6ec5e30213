// ks_lanes.hpp -- sums over the 64 lanes of a wavefront through register
// exchanges (v_permlane32_swap / v_permlane16_swap between the halves and
// rows, DPP inside a row of 16), without the LDS crossbar that __shfl uses.
// Every sum here adds in the same tree (lane pairs i ^ 32, i ^ 16, i ^ 15,
// i ^ 7, i ^ 2, i ^ 1), so a value's sum does not depend on how many sums are
// formed together.
#pragma once

#include "ks_common.hpp"

namespace ks {

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140;

template <int CTRL>
__device__ __forceinline__ double dpp_(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, true));
}

// a' = (a of the lower half, b of the lower half), b' = (a upper, b upper): the
// sum a' + b' is a summed over the halves in the lower lanes, b in the upper ones
__device__ __forceinline__ double sum32(double a, double b) {
    const u32x2 l = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const u32x2 h = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double(h.x, l.x) + __hiloint2double(h.y, l.y);
}
// the same between the even and the odd rows of 16 lanes
__device__ __forceinline__ double sum16(double a, double b) {
    const u32x2 l = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const u32x2 h = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double(h.x, l.x) + __hiloint2double(h.y, l.y);
}
__device__ __forceinline__ double sum8(double a, double b, bool up) {
    return pick(up, b, a) + dpp_<DPP_MIRROR>(pick(up, a, b));
}
__device__ __forceinline__ double sum4(double a, double b, bool up) {
    return pick(up, b, a) + dpp_<DPP_HALF_MIRROR>(pick(up, a, b));
}
__device__ __forceinline__ double sum8(double v) { return v + dpp_<DPP_MIRROR>(v); }
__device__ __forceinline__ double sum4(double v) { return v + dpp_<DPP_HALF_MIRROR>(v); }
__device__ __forceinline__ double sum21(double v) {
    v += dpp_<DPP_XOR2>(v);
    return v + dpp_<DPP_XOR1>(v);
}

__device__ __forceinline__ cplx sum32(cplx a, cplx b) { return mk(sum32(a.x, b.x), sum32(a.y, b.y)); }
__device__ __forceinline__ cplx sum16(cplx a, cplx b) { return mk(sum16(a.x, b.x), sum16(a.y, b.y)); }
__device__ __forceinline__ cplx sum8(cplx a, cplx b, bool u) { return mk(sum8(a.x, b.x, u), sum8(a.y, b.y, u)); }
__device__ __forceinline__ cplx sum4(cplx a, cplx b, bool u) { return mk(sum4(a.x, b.x, u), sum4(a.y, b.y, u)); }
__device__ __forceinline__ cplx sum8(cplx v) { return mk(sum8(v.x), sum8(v.y)); }
__device__ __forceinline__ cplx sum4(cplx v) { return mk(sum4(v.x), sum4(v.y)); }
__device__ __forceinline__ cplx sum21(cplx v) { return mk(sum21(v.x), sum21(v.y)); }

// The sum of v over the wavefront, in every lane.
template <typename T>
__device__ __forceinline__ T lane_sum(T v) {
    v = sum32(v, v);
    v = sum16(v, v);
    return sum21(sum4(sum8(v)));
}

// The value of lane l (uniform) in every lane.
__device__ __forceinline__ double lane_get(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}
__device__ __forceinline__ cplx lane_get(cplx v, int l) { return mk(lane_get(v.x, l), lane_get(v.y, l)); }

// The sums of R values over the wavefront at once: lane l ends with the sum of
// value l / (64 / R).
template <typename T>
__device__ __forceinline__ T lane_sums(const T (&r)[16], int lane) {
    T a[8], b[4], c[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = sum32(r[i], r[i + 8]);
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = sum16(a[i], a[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; ++i) c[i] = sum8(b[i], b[i + 2], lane & 8);
    return sum21(sum4(c[0], c[1], lane & 4));
}
template <typename T>
__device__ __forceinline__ T lane_sums(const T (&r)[8], int lane) {
    T a[4], b[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = sum32(r[i], r[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; ++i) b[i] = sum16(a[i], a[i + 2]);
    return sum21(sum4(sum8(b[0], b[1], lane & 8)));
}
template <typename T>
__device__ __forceinline__ T lane_sums(const T (&r)[4], int lane) {
    T a[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = sum32(r[i], r[i + 2]);
    return sum21(sum4(sum8(sum16(a[0], a[1]))));
}

}  // namespace ks
