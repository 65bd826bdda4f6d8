// Routing helpers shared by the top-k kernels (one 64-lane wavefront per
// token; expert e = lane + 64 i sits in register i of its lane).
//
// A token's few hundred instructions run once, so these kernels are bound by
// latency: instruction fetch (cold at every launch) and dependent lane
// operations.  Hence 32-bit keys (one DPP instruction per reduction step where
// a 64-bit key with the index took six) and ties resolved with ballots.
#pragma once

#include <type_traits>

#include "device.hpp"

namespace ecospec {

// Position of a value in the routing order as an unsigned integer: larger
// first, -0 with +0, NaN (1) after every number (-inf is 0x007fffff); 0 is
// left for "not eligible".
__device__ __forceinline__ uint32_t rank_key(float v)
{
    uint32_t b = __float_as_uint(v);
    if (v != v) return 1u;
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// The value of a key (1 gives a NaN).
__device__ __forceinline__ float key_value(uint32_t key)
{
    return __uint_as_float((key & 0x80000000u) ? key ^ 0x80000000u : ~key);
}

// Maximum over the wavefront, as a uniform value (DPP row shifts and broadcasts: lane 63 ends with it).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_max_step(uint32_t v)
{
    const uint32_t o = __builtin_amdgcn_update_dpp(0u, v, CTRL, ROW_MASK, 0xf, false);
    return o > v ? o : v;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    v = dpp_max_step<0x111, 0xf>(v);  // row_shr:1
    v = dpp_max_step<0x112, 0xf>(v);  // row_shr:2
    v = dpp_max_step<0x114, 0xf>(v);  // row_shr:4
    v = dpp_max_step<0x118, 0xf>(v);  // row_shr:8
    v = dpp_max_step<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_max_step<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(v, 63);
}

// k rounds of a wave-wide maximum over the experts' keys (0 = not eligible),
// equal keys by the lower expert: lane r returns the expert of rank r, and its
// key in *key_out.
template <int EPL>
__device__ __forceinline__ int select_ranks(uint32_t (&key)[EPL], int k, uint32_t *key_out)
{
    const int lane = lane_id();
    int mine = -1;
    uint32_t mkey = 0u;
    for (int r = 0; r < k; ++r) {
        uint32_t best = key[0];
#pragma unroll
        for (int i = 1; i < EPL; ++i) best = key[i] > best ? key[i] : best;
        const uint32_t win = wave_max_u32(best);
        int e = -1;  // lowest expert holding it
#pragma unroll
        for (int i = EPL - 1; i >= 0; --i) {
            const uint64_t m = __ballot(key[i] == win);
            if (m) e = kWave * i + (int)__builtin_ctzll(m);
        }
#pragma unroll
        for (int i = 0; i < EPL; ++i)
            if (lane + kWave * i == e) key[i] = 0u;
        if (lane == r) {
            mine = e;
            mkey = win;
        }
    }
    *key_out = mkey;
    return mine;
}

// val of expert `mine` (held by lane mine % 64 in register mine / 64).  Call
// it from every lane: a lane-permute reads nothing from inactive lanes.
template <int EPL>
__device__ __forceinline__ float value_of(const float (&val)[EPL], int mine)
{
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const float c = __shfl(val[i], (mine - kWave * i) & (kWave - 1), kWave);
        if (mine >= kWave * i && mine < kWave * (i + 1)) v = c;
    }
    return v;
}

// Sum of a value held by lanes 0 .. k-1 (0 elsewhere), in those lanes: the butterfly of wave_sum, pairing
// lanes 32, 16, 8, ... 1 apart, with the steps within a row of 16 as DPP rotations (the same sums, since
// every step leaves its values periodic) and the two wider steps left out where they add zeros.
__device__ __forceinline__ float rank_sum(float v, int k)
{
    if (k > 32) v += __shfl_xor(v, 32, kWave);
    if (k > 16) v += __shfl_xor(v, 16, kWave);
    auto ror = [](float x, auto ctrl) {
        return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), decltype(ctrl)::value, 0xf, 0xf, false));
    };
    v += ror(v, std::integral_constant<int, 0x128>{});  // row_ror:8
    v += ror(v, std::integral_constant<int, 0x124>{});
    v += ror(v, std::integral_constant<int, 0x122>{});
    v += ror(v, std::integral_constant<int, 0x121>{});
    return v;
}

// Gate weight of rank `lane` (< k) from its logit v, held one per lane: a
// softmax over the k selected logits (score 0; rank 0 holds the largest) or a
// renormalised sigmoid (score 1), in fp32.  Every lane must call it.
__device__ __forceinline__ float gate_weight(float v, int k, int score)
{
    const bool sel = lane_id() < k;
    if (!sel) v = 0.f;
    const float m = score == 0 ? __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))) : 0.f;
    const float x = expf(score == 0 ? v - m : -v);
    const float g = !sel ? 0.f : score == 0 ? x : 1.f / (1.f + x);
    return g / rank_sum(g, k);
}

}  // namespace ecospec
