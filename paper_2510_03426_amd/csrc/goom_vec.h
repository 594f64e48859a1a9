// Helpers of the matrix-vector kernels (goom_vec.hip, goom_vec_adjoint.hip): reductions over the sixteen lanes that share a row, and
// the conversion of a GOOM entry on a given power of two.
#pragma once
#include "goom_chain_kernel.h"

#include <type_traits>

namespace goom_chain {

namespace {

template <int CTRL> __device__ inline float dpp_of(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ inline double dpp_of(double v)
{
    const u2 b = __builtin_bit_cast(u2, v);
    u2 r;
    r[0] = (unsigned)__builtin_amdgcn_mov_dpp((int)b[0], CTRL, 0xF, 0xF, true);
    r[1] = (unsigned)__builtin_amdgcn_mov_dpp((int)b[1], CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, r);
}
__device__ inline float raw_max(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ inline double raw_max(double a, double b) { return __builtin_fmax(a, b); }
// sum / maximum over the sixteen lanes of a row (in every one of them)
template <typename V> __device__ inline V sum16(V v)
{
    v += dpp_of<0xB1>(v);
    v += dpp_of<0x4E>(v);
    v += dpp_of<0x141>(v);
    v += dpp_of<0x140>(v);
    return v;
}
template <typename V> __device__ inline V max16(V v)
{
    v = raw_max(v, dpp_of<0xB1>(v));
    v = raw_max(v, dpp_of<0x4E>(v));
    v = raw_max(v, dpp_of<0x141>(v));
    v = raw_max(v, dpp_of<0x140>(v));
    return v;
}

// (+-) 2^(re log2(e) - n), one rounding of a small argument; -inf gives zero, NaN stays NaN
__device__ inline float scaled_entry(float re, float im, float n)
{
    const float kHi = 1.44269502162933349609375f; // float nearest log2(e)
    const float kLo = 1.925963033500011e-8f;      // log2(e) - kHi
    float t = __builtin_fmaf(re, kHi, -n);
    t = __builtin_fmaf(re, kLo, t);
    return Comp<float>::apply_sign(__builtin_amdgcn_exp2f(t), im);
}
__device__ inline double scaled_entry(double re, double im, double n)
{
    const double t = __builtin_fma(re, kLog2e, -n);
    const double k = __builtin_rint(t);
    const double y = __builtin_ldexp(Comp<double>::exp2_small(t - k), (int)(k < -4000.0 ? -4000.0 : k));
    return Comp<double>::apply_sign(t < -1200.0 ? 0.0 : y, im);
}

constexpr float kNone = -1.0e30f; // stands for the exponent of zero

} // namespace

} // namespace goom_chain
