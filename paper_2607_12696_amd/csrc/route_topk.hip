// Router top-k on gfx950: one 64-lane wavefront per token.
//
// Each token's E logits (E <= 1024) are spread over the lanes of one wave.
// k rounds of a wave-wide maximum over order-preserving 32-bit keys pick the
// experts in routing order (-0 with +0, NaN below every number, equal logits
// by the lower index); the winner's key is cleared after each round.  Gate
// weights are then a softmax or a renormalised sigmoid over the k selected
// logits, held one per lane, in fp32.
#include "device.hpp"
#include "launch.hpp"
#include "route_common.hpp"

namespace ecospec {

// slices == 0: `logits` is [T][E].  slices > 0: `logits` holds the router's
// K-slice partial sums [slices][T][E], added here in slice order; the sums
// are also stored to logits_out when it is given.
template <int EPL>  // experts per lane: ceil(E / 64)
__global__ __launch_bounds__(256) void route_topk_kernel(const float *__restrict__ logits, int slices, int T, int E,
                                                         int k, int score, int32_t *__restrict__ topk_idx,
                                                         float *__restrict__ topk_w, float *__restrict__ logits_out)
{
    const int lane = lane_id();
    const int t = blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
    if (t >= T) return;  // uniform per wave
    const float *row = logits + (size_t)t * E;

    float val[EPL];
    if (slices == 0) {
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const int e = lane + kWave * i;
            val[i] = e < E ? row[e] : 0.f;
        }
    } else {
        // Sum the slices in order, a chunk at a time with all its loads in flight: 16 slices up to 4 experts per
        // lane (a d of 8192 is one round trip), 8 where there are no more.  Loads past the last slice or expert
        // read zeros, and a chunk has a descriptor of its own, so that its offsets stay below 2^31.
        const size_t te = (size_t)T * E;
        constexpr int MOST = EPL <= 4 ? 16 : EPL < 8 ? 8 : 2;
#pragma unroll
        for (int i = 0; i < EPL; ++i) val[i] = 0.f;
        auto add_chunk = [&](int s0, auto width) {
            constexpr int CH = decltype(width)::value;
            const rsrc_t rp = make_rsrc(logits + s0 * te, (uint32_t)(min(CH, slices - s0) * te * 4));
            float p[EPL][CH];
#pragma unroll
            for (int i = 0; i < EPL; ++i) {
                const int e = lane + kWave * i;
                const uint32_t off = e < E ? ((uint32_t)t * (uint32_t)E + (uint32_t)e) * 4u : kOff;
#pragma unroll
                for (int c = 0; c < CH; ++c)
                    p[i][c] = __uint_as_float(
                        __builtin_amdgcn_raw_buffer_load_b32(rp, (int)(off + (uint32_t)c * (uint32_t)te * 4u), 0, 0));
            }
            __builtin_amdgcn_sched_barrier(0);  // keep every load ahead of the first sum
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int i = 0; i < EPL; ++i) val[i] += p[i][c];  // zeros past the last slice
        };
        if (te < (1u << 29) / MOST) {
            if (MOST == 16 && slices <= 8)
                add_chunk(0, std::integral_constant<int, 8>{});
            else
                for (int s0 = 0; s0 < slices; s0 += MOST) add_chunk(s0, std::integral_constant<int, MOST>{});
        } else {  // partial sums of 2 GiB and more a chunk: a slice at a time
#pragma unroll 1
            for (int c = 0; c < slices; ++c)
#pragma unroll
                for (int i = 0; i < EPL; ++i) {
                    const int e = lane + kWave * i;
                    if (e < E) val[i] += logits[((size_t)c * T + t) * E + e];
                }
        }
        if (logits_out) {
#pragma unroll
            for (int i = 0; i < EPL; ++i) {
                const int e = lane + kWave * i;
                if (e < E) logits_out[(size_t)t * E + e] = val[i];
            }
        }
    }
    uint32_t key[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) key[i] = lane + kWave * i < E ? rank_key(val[i]) : 0u;
    uint32_t mkey;
    const int mine = select_ranks(key, k, &mkey);
    const float wgt = gate_weight(key_value(mkey), k, score);
    if (lane < k) {
        topk_idx[(size_t)t * k + lane] = mine;
        topk_w[(size_t)t * k + lane] = wgt;
    }
}

// Group-limited routing (the DeepSeek-V3 rule): sigmoid scores s, choice
// scores c = s + bias; the E experts form G contiguous groups of gs = E / G
// (gs >= 2); a group's score is the sum of its two highest choice scores (in
// the routing order of rank_key, so NaN only counts when a group has fewer
// than two numbers); the TG groups of highest score (ties: lower group) stay
// eligible and the k highest choice scores among their experts are selected,
// in order.  Gate weights: scale * s / sum(s) over the selected.  One
// wavefront per token; the choice scores go through LDS so that lane g can
// score group g.
template <int EPL>
__global__ __launch_bounds__(256) void route_grouped_kernel(const float *__restrict__ logits,
                                                            const float *__restrict__ bias, int T, int E, int k,
                                                            int G, int TG, float scale, int32_t *__restrict__ topk_idx,
                                                            float *__restrict__ topk_w)
{
    __shared__ uint32_t cs[4][1024];
    const int lane = lane_id(), wv = threadIdx.x / kWave;
    const int t = blockIdx.x * 4 + wv;
    const bool active = t < T;
    const int gs = E / G;
    float sv[EPL];
    uint32_t key[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int e = lane + kWave * i;
        const float l = (active && e < E) ? logits[(size_t)t * E + e] : 0.f;
        sv[i] = 1.f / (1.f + expf(-l));
        key[i] = rank_key(sv[i] + ((bias && e < E) ? bias[e] : 0.f));
        if (e < E) cs[wv][e] = key[i];
    }
    __syncthreads();
    if (!active) return;  // uniform per wave, after the block's only barrier

    // The two highest keys of each group: 1 << sh lanes per group take every (1 << sh)-th expert of it (8 lanes for
    // 8 groups; one lane a group, walking its 32 experts, took 4 us of the kernel's 12), then merge.
    const int sh = 31 - __clz(kWave / G);
    const int grp = lane >> sh, sub = lane & ((1 << sh) - 1);
    uint32_t k1 = 0u, k2 = 0u;
    if (grp < G)
        for (int j = sub; j < gs; j += 1 << sh) {
            const uint32_t kv = cs[wv][grp * gs + j];
            k2 = max(k2, min(k1, kv));
            k1 = max(k1, kv);
        }
    for (int m = 1; m < (1 << sh); m <<= 1) {
        const uint32_t o1 = __shfl_xor(k1, m, kWave), o2 = __shfl_xor(k2, m, kWave);
        k2 = max(max(k2, o2), min(k1, o1));
        k1 = max(k1, o1);
    }
    uint32_t gkey = grp < G && sub == 0 ? rank_key(key_value(k1) + key_value(k2)) : 0u;
    uint64_t gmask = 0ull;  // bit g: group g stays eligible
    for (int r = 0; r < TG; ++r) {
        const uint32_t win = wave_max_u32(gkey);
        const int first = (int)__builtin_ctzll(__ballot(gkey == win));  // the lowest group of that score
        gmask |= 1ull << (first >> sh);
        if (lane == first) gkey = 0u;
    }
    const float inv = 1.f / (float)gs;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int e = lane + kWave * i;
        const int g = (int)(((float)e + 0.5f) * inv);  // e / gs: exact for e < 1024
        if (!(e < E && ((gmask >> g) & 1ull))) key[i] = 0u;
    }
    uint32_t mkey;
    const int mine = select_ranks(key, k, &mkey);
    const bool sel = lane < k;
    const float sm = value_of(sv, mine);  // every lane takes part in the shuffles
    const float g = sel ? sm : 0.f;
    const float sum = rank_sum(g, k);
    if (sel) {
        topk_idx[(size_t)t * k + lane] = mine;
        topk_w[(size_t)t * k + lane] = scale * (g / sum);
    }
}

hipError_t launch_route_grouped(const float *logits, const float *bias, int T, int E, int k, int G, int TG,
                                float scale, int32_t *idx, float *w, hipStream_t stream)
{
    const dim3 block(256), grid((T + 3) / 4);
    const int epl = (E + kWave - 1) / kWave;
#define GROUPED_CASE(N)                                                                                         \
    case N:                                                                                                     \
        hipLaunchKernelGGL(route_grouped_kernel<N>, grid, block, 0, stream, logits, bias, T, E, k, G, TG, scale, \
                           idx, w);                                                                             \
        break;
    switch (epl) {
        GROUPED_CASE(1) GROUPED_CASE(2) GROUPED_CASE(3) GROUPED_CASE(4) GROUPED_CASE(5) GROUPED_CASE(6)
        GROUPED_CASE(7) GROUPED_CASE(8) GROUPED_CASE(9) GROUPED_CASE(10) GROUPED_CASE(11) GROUPED_CASE(12)
        GROUPED_CASE(13) GROUPED_CASE(14) GROUPED_CASE(15) GROUPED_CASE(16)
    default: return hipErrorInvalidValue;
    }
#undef GROUPED_CASE
    return hipGetLastError();
}

hipError_t launch_route_topk(const float *logits, int slices, int T, int E, int k, int score, int32_t *idx, float *w,
                             float *logits_out, hipStream_t stream)
{
    const dim3 block(256), grid((T + 3) / 4);
    const int epl = (E + kWave - 1) / kWave;
#define ROUTE_CASE(N)                                                                                          \
    case N:                                                                                                    \
        hipLaunchKernelGGL(route_topk_kernel<N>, grid, block, 0, stream, logits, slices, T, E, k, score, idx, w, \
                           logits_out);                                                                        \
        break;
    switch (epl) {
        ROUTE_CASE(1) ROUTE_CASE(2) ROUTE_CASE(3) ROUTE_CASE(4) ROUTE_CASE(5) ROUTE_CASE(6) ROUTE_CASE(7)
        ROUTE_CASE(8) ROUTE_CASE(9) ROUTE_CASE(10) ROUTE_CASE(11) ROUTE_CASE(12) ROUTE_CASE(13)
        ROUTE_CASE(14) ROUTE_CASE(15) ROUTE_CASE(16)
    default: return hipErrorInvalidValue;
    }
#undef ROUTE_CASE
    return hipGetLastError();
}

}  // namespace ecospec
