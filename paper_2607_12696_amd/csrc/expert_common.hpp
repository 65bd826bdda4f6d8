// What the expert kernels share: the weight formats' operand layouts and
// decoding, and the activation between the two projections.
#pragma once

#include "device.hpp"
#include "launch.hpp"

namespace ecospec {

enum { FMT_BF16 = 0, FMT_FP8 = 1, FMT_MXFP4 = 2 };

constexpr int kMacroK = 128;            // reduction elements per macro step
constexpr int kAuxNT = 2;               // nontemporal: streamed weights should not displace activations

// kVecs: 16-byte vectors per lane in one 16 x 128 block of a tile; kBlocks:
// 128-wide K blocks per macro step.  MXFP4 takes two blocks a step, so that a
// step streams 2 KiB per tile like FP8 and pays its fixed per-step work (the
// activation staging, the barrier, the item bookkeeping) over as many bytes.
template <int FMT> struct Fmt;
template <> struct Fmt<FMT_BF16>  { static constexpr int kVecs = 4, kBlocks = 1; };
template <> struct Fmt<FMT_FP8>   { static constexpr int kVecs = 2, kBlocks = 1; };
template <> struct Fmt<FMT_MXFP4> { static constexpr int kVecs = 1, kBlocks = 2; };

// The scale operand of the scaled conversions (v_cvt_scalef32_*): the
// instruction takes the operand's exponent field as an e8m0 code, so field 0
// scales by 2^-127 and field 255 gives NaN, as the OCP MX definition of the
// code does (checked on the device against the exact scale value for all 256
// codes and all 256 FP4 code pairs: identical results).  The code shifted into
// the exponent field is therefore the operand for every code, with no special
// cases.
__device__ __forceinline__ float e8m0_scale_operand(uint32_t code) { return __uint_as_float((code & 0xffu) << 23); }

// bf16 A operand of sub-step s (0 .. 3; the lane's weights 8s .. 8s+7 of one
// 16 x 128 block, v: its vectors).
// Exact: FP8 codes as they are (the converter's scale operand only takes a
// power of two, so the 128x128 block scale multiplies the fp32 partial sum of
// the step instead); MXFP4 codes times sc, their 2^e8m0 group scale.
template <int FMT>
__device__ __forceinline__ bf16x8 decode8(const u32x4 *v, int s, float sc)
{
    if constexpr (FMT == FMT_BF16) {
        return __builtin_bit_cast(bf16x8, v[s]);
    } else if constexpr (FMT == FMT_FP8) {
        const uint32_t w0 = v[s >> 1][(s & 1) * 2], w1 = v[s >> 1][(s & 1) * 2 + 1];
        u32x4 o;
        o[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, false));
        o[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, true));
        o[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, false));
        o[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, true));
        return __builtin_bit_cast(bf16x8, o);
    } else {
        const uint32_t w = v[0][s];
        u32x4 o;
        o[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, sc, 0));
        o[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, sc, 1));
        o[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, sc, 2));
        o[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, sc, 3));
        return __builtin_bit_cast(bf16x8, o);
    }
}

// g * sigmoid(s * g) with the hardware exp2 and reciprocal (about 2 ulp in
// fp32, far below the bf16 rounding of H): g / (1 + e^(-s g)).  Large -s g
// gives 1 + inf, whose reciprocal is 0, and NaN stays NaN, as in the
// division form.
__device__ __forceinline__ float gated(float g, float s)
{
    return g * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-s * g * 1.44269504088896341f));
}

// h from the gate and up values of one row (biases already added):
// act 0 silu(g) * u; act 1 (GPT-OSS) with g capped at limit and u clamped to
// [-limit, limit], g * sigmoid(alpha * g) * (u + 1).  The comparisons keep NaN.
__device__ __forceinline__ float activate(int act, float alpha, float limit, float g, float u)
{
    if (act == 0) return gated(g, 1.f) * u;
    if (g > limit) g = limit;
    if (u > limit) u = limit;
    if (u < -limit) u = -limit;
    return gated(g, alpha) * (u + 1.f);
}

__device__ __forceinline__ float activate(const VerifyArgs &a, float g, float u)
{
    return activate(a.act, a.alpha, a.limit, g, u);
}

}  // namespace ecospec
