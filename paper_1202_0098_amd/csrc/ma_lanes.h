// Exchanges between the lanes of a wavefront in registers (gfx950): DPP
// within rows of 16 lanes, v_permlane16_swap and v_permlane32_swap between
// them.  None touches LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace ma {

namespace {

typedef unsigned uint2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double join(unsigned lo, unsigned hi)
{
    return __hiloint2double((int)hi, (int)lo);
}

// v of the lane that the DPP control names (every lane enabled)
template <int CTRL>
__device__ __forceinline__ double dpp(double v)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false));
}

constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;            // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;  // lane 7 - l of 8, 15 - l of 16
constexpr int kDppRor8 = 0x128;                            // lane l ^ 8 of 16

// a: lanes of the even rows (lower half) of a, then those of b; b: the odd
// rows (upper half) of both.  The sum of the two is the exchange step of a
// transposed reduction over lane bit 4 (5): a's total in the even rows (lower
// half), b's in the others.
__device__ __forceinline__ void swap16(double &a, double &b)
{
    const uint2v l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a),
                                                      (unsigned)__double2loint(b), false, false);
    const uint2v h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a),
                                                      (unsigned)__double2hiint(b), false, false);
    a = join(l.x, h.x);
    b = join(l.y, h.y);
}

__device__ __forceinline__ void swap32(double &a, double &b)
{
    const uint2v l = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a),
                                                      (unsigned)__double2loint(b), false, false);
    const uint2v h = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a),
                                                      (unsigned)__double2hiint(b), false, false);
    a = join(l.x, h.x);
    b = join(l.y, h.y);
}

__device__ __forceinline__ double add_xor16(double v)
{
    double w = v;
    swap16(v, w);
    return v + w;
}

__device__ __forceinline__ double add_xor32(double v)
{
    double w = v;
    swap32(v, w);
    return v + w;
}

// sum over each aligned group of W lanes (16, 32 or 64), in every lane
template <int W>
__device__ __forceinline__ double sum_within(double v)
{
    v += dpp<kDppXor1>(v);
    v += dpp<kDppXor2>(v);
    v += dpp<kDppHalfMirror>(v);
    v += dpp<kDppMirror>(v);
    if constexpr (W >= 32) v = add_xor16(v);
    if constexpr (W >= 64) v = add_xor32(v);
    return v;
}

// sum over the lanes that agree modulo W (16, 32 or 64), in every lane
template <int W>
__device__ __forceinline__ double sum_across(double v)
{
    if constexpr (W <= 16) v = add_xor16(v);
    if constexpr (W <= 32) v = add_xor32(v);
    return v;
}

// a value that every lane holds, as a scalar
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Transposed reduction of eight values per lane over the wavefront:
// afterwards v[0] of lane l holds the total of value tr_index<8>(l).  The two
// widest exchanges, most of the work, are lane swaps without selects.
__device__ __forceinline__ void lane_reduce8(double (&v)[8])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        swap32(v[k], v[k + 4]);
        v[k] += v[k + 4];
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        swap16(v[k], v[k + 2]);
        v[k] += v[k + 2];
    }
    const bool hi = (threadIdx.x & 8) != 0;
    const double send = hi ? v[0] : v[1], keep = hi ? v[1] : v[0];
    v[0] = keep + dpp<kDppRor8>(send);
    v[0] += dpp<kDppHalfMirror>(v[0]);
    v[0] += dpp<kDppXor2>(v[0]);
    v[0] += dpp<kDppXor1>(v[0]);
}

// 1 / sqrt(x) for normal x > 0: v_rsq_f64 (about 1e-8) and one third-order
// correction, within 2 ulp
__device__ __forceinline__ double rsqrt_fast(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// 1 / x for normal x: v_rcp_f64 and two Newton steps
__device__ __forceinline__ double rcp_fast(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

}  // namespace

}  // namespace ma
