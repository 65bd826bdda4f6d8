// Conversion of expert weights from the interchange layout ([E][N][K], K
// contiguous) to the streaming layout the verify kernels read.
//
// Streaming layout of one N x K matrix (N % 16 == 0; K padded to Kp, the next
// multiple of 128, with zero codes): blocks of 16 rows x 128 reduction
// elements, block (rb, kb) at byte offset (rb * Kp/128 + kb) * B where B is
// 4096 (bf16), 2048 (FP8) or 1024 (MXFP4) bytes.  A block is B/1024 vectors
// of 1 KiB; in vector i, the 16 bytes at offset 16*l (l = c + 16*g, c < 16,
// g < 4) hold the weights of row rb*16 + c starting at element
// kb*128 + 32*g + i*(32*1024/B).  So lane l of a wavefront reading vector i
// with one 16-byte load gets exactly the A-operand fragment of the matrix-core
// instruction, and a wavefront reads each vector as 1 KiB of contiguous memory.
//
// W_gate and W_up can also be packed as one pair (moe_pack_gate_up): block
// (rb, kb) of the pair is the gate block followed by the up block, so a
// wavefront reads both tiles of a step as one contiguous run (one stream
// instead of two, measured 4% more bandwidth in the kernel's geometry).
// W_down likewise (moe_pack_down): row tiles 2p and 2p + 1 (the two tiles of
// one down wavefront) are interleaved block by block, block (2p + j, kb) at
// ((p * Kp/128 + kb) * 2 + j) * B.
//
// MXFP4 scales move to the same blocking, four blocks to a 256-byte quad: in
// quad q of row tile rb, the 4 bytes at offset 4*l (l = c + 16*g) are the
// e8m0 codes of row rb*16 + c for the 32-element chunks (4q + j)*4 + g,
// j = 0..3 (127, i.e. 1.0, in the padding), so one dword load per lane
// brings a lane's codes for four blocks.  FP8 block scales keep their
// [N/128][K/128] layout.
#include <type_traits>

#include "device.hpp"
#include "launch.hpp"

namespace ecospec {

// Bound by memory: every byte is read and written once.  A wavefront takes runs
// of kPackRun blocks along K of one 16-row tile of one expert (of W_gate and of
// W_up where they are packed as a pair: the pair's blocks are then written side
// by side).  So it reads whole lines of its rows (128 elements and more) with all
// of a run's loads in flight, writes each vector as 1 KiB, and divides nothing
// per vector.  The stores are non-temporal: the packed weights are next read in a
// verification, long after.  The scales go with their blocks (a run is the quad
// of the MXFP4 scale layout), so a pair of matrices is one launch.  Against a
// thread per vector with its own index divisions and scales in launches of their
// own (time of a layer's share): 64 DeepSeek FP8 experts 1108 -> 1016 us (5.6 TB/s
// read and written), 32 GPT-OSS MXFP4 experts 228 -> 158 us, 4 DeepSeek experts 79 ->
// 55 us, 8 Qwen bf16 experts 116 -> 110 us.
// Gate and up by different workgroups measured 1284 us for the first of these;
// 128 threads 5% slower, 256 to 1024 and runs of 2 to 4 within 4%.
constexpr int kPackRun = 4;
constexpr int kPackWaves = 8;

struct PackMatrix {
    const uint8_t *w, *s;
    uint8_t *s_out;
};

struct PackArgs {
    PackMatrix m[2];  // gate and up, or one matrix
    uint8_t *dst;
    size_t row_bytes;   // of a row of w
    size_t src_mat, dst_mat, s_mat, s_out_mat;  // bytes from one expert's matrix / scales to the next
    size_t row_tiles;   // E * N / 16
    int tiles, nkb, K, fmt;
    size_t t_step;      // tiles from one turn to the next of a workgroup
    int wave_tiles;     // a tile per wavefront; else the workgroups of a column of the grid share one
    int waves, kb_step; // wavefronts of a workgroup; blocks from one run to the next of a wavefront
    int tile_pairs;
};

// The scales of the run from block kb0 on of row tile rb of expert e.  Byte by byte where alignment is not given.
__device__ __forceinline__ void pack_scales(const PackArgs &P, const PackMatrix &m, size_t e, int rb, int kb0)
{
    const int lane = lane_id();
    if (P.fmt == 1) {  // FP8 block scales, [N/128][K/128] as they are: copied with the first tile of each 128 rows
        if ((rb & 7) == 0 && lane < kPackRun && kb0 + lane < P.nkb) {
            const size_t o = ((size_t)(rb >> 3) * P.nkb + kb0 + lane) * 4;
            __builtin_memcpy(m.s_out + e * P.s_out_mat + o, m.s + e * P.s_mat + o, 4);
        }
    } else if (P.fmt == 2) {  // MXFP4: [ceil(Kp/512)][64][4] of this tile, a dword (four blocks' codes) per lane
        const int nq = (P.nkb + 3) / 4, chunks = P.K / 32, base = kb0 * 4 + (lane >> 4);
        const uint8_t *row = m.s + e * P.s_mat + (size_t)(rb * 16 + (lane & 15)) * chunks;
        uint8_t code[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) code[j] = base + 4 * j < chunks ? row[base + 4 * j] : (uint8_t)127;
        __builtin_memcpy(m.s_out + e * P.s_out_mat + (((size_t)rb * nq + kb0 / 4) * 64 + lane) * 4, code, 4);
    }
}

template <int VECS, int NM>
__global__ __launch_bounds__(kPackWaves *kWave) void pack_kernel(PackArgs P)
{
    constexpr uint32_t B = VECS * 1024u;
    static_assert(kPackRun == 4, "a run is a quad of the MXFP4 scales");
    const int lane = lane_id(), c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int kb_first = P.wave_tiles ? 0 : ((int)blockIdx.y * P.waves + wave) * kPackRun;
    for (size_t t = P.wave_tiles ? (size_t)blockIdx.x * P.waves + wave : blockIdx.x; t < P.row_tiles; t += P.t_step) {
        const size_t e = t / (size_t)P.tiles;
        const int rb = (int)(t - e * (size_t)P.tiles);
        const size_t soff = e * P.src_mat + (size_t)(rb * 16 + c) * P.row_bytes + (size_t)g * (VECS * 16);
        const size_t first = P.tile_pairs ? (size_t)(rb >> 1) * P.nkb * 2 + (rb & 1) : (size_t)rb * P.nkb * NM;
        const size_t step = (P.tile_pairs || NM == 2 ? 2 : 1) * (size_t)B;
        uint8_t *dst = P.dst + e * P.dst_mat + first * B + (size_t)lane * 16;
        for (int kb0 = kb_first; kb0 < P.nkb; kb0 += P.kb_step) {
            u32x4 v[kPackRun][NM][VECS];
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int r = 0; r < kPackRun; ++r) {
                    const int kb = kb0 + r;
                    const bool in = kb < P.nkb && kb * 128 + 32 * g < P.K;  // K % 32 == 0: a chunk is all in or all out
#pragma unroll
                    for (int i = 0; i < VECS; ++i)
                        v[r][m][i] = in ? *reinterpret_cast<const u32x4 *>(P.m[m].w + soff + (size_t)kb * (VECS * 64) + 16 * i)
                                        : u32x4{0u, 0u, 0u, 0u};
                }
#pragma unroll
            for (int r = 0; r < kPackRun; ++r)
                if (kb0 + r < P.nkb)
#pragma unroll
                    for (int m = 0; m < NM; ++m)
#pragma unroll
                        for (int i = 0; i < VECS; ++i)
                            __builtin_nontemporal_store(
                                v[r][m][i], reinterpret_cast<u32x4 *>(dst + (size_t)(kb0 + r) * step + m * B + 1024 * i));
        }
        if (P.fmt == 0) continue;
        for (int kb0 = kb_first; kb0 < P.nkb; kb0 += P.kb_step)
#pragma unroll
            for (int i = 0; i < NM; ++i) pack_scales(P, P.m[i], e, rb, kb0);
    }
}

size_t packed_matrix_bytes(int fmt, int N, int K)
{
    const size_t kp = (size_t)((K + 127) / 128) * 128;
    return fmt == 0 ? (size_t)N * kp * 2 : fmt == 1 ? (size_t)N * kp : (size_t)N * kp / 2;
}

size_t packed_scale_bytes(int fmt, int N, int K)
{
    if (fmt == 1) return (size_t)(N / 128) * (K / 128) * 4;
    if (fmt == 2) return (size_t)N * (((K + 127) / 128 + 3) / 4) * 16;
    return 0;
}

// One or two (wu: gate and up as a pair) stacked matrices into wp.
static hipError_t pack(int fmt, int E, int N, int K, const void *w, const void *s, const void *wu, const void *su, void *wp,
                       void *sp, void *sup, int tile_pairs, hipStream_t stream)
{
    PackArgs a{};
    a.m[0] = PackMatrix{static_cast<const uint8_t *>(w), static_cast<const uint8_t *>(s), static_cast<uint8_t *>(sp)};
    a.m[1] = PackMatrix{static_cast<const uint8_t *>(wu), static_cast<const uint8_t *>(su), static_cast<uint8_t *>(sup)};
    a.dst = static_cast<uint8_t *>(wp);
    const bool pair = wu != nullptr;
    a.tile_pairs = tile_pairs;
    a.fmt = fmt;
    a.K = K;
    a.nkb = (K + 127) / 128;
    a.tiles = N / 16;
    a.row_tiles = (size_t)E * a.tiles;
    a.row_bytes = fmt == 0 ? (size_t)K * 2 : fmt == 1 ? (size_t)K : (size_t)K / 2;
    a.src_mat = a.row_bytes * N;
    a.dst_mat = packed_matrix_bytes(fmt, N, K) * (pair ? 2 : 1);
    a.s_mat = fmt == 2 ? (size_t)N * (K / 32) : packed_scale_bytes(fmt, N, K);
    a.s_out_mat = packed_scale_bytes(fmt, N, K);
    // As a rule a workgroup of eight wavefronts takes a tile.  Tiles of up to 4 KiB are a wavefront's each, since a
    // workgroup's start costs more than such a tile (K = 128, 512 MiB read and written: bf16 93 us with a thread per vector,
    // 114 with a workgroup a tile, 73 with a wavefront; MXFP4 219, 353, 107; from 8 KiB on a workgroup is as fast or
    // faster: bf16 pairs, K = 256, 166 us against 181).  Where there are no more tiles than compute units, a tile's runs
    // are spread over workgroups of one wavefront (bf16 128 x 8192: 4.4, 11.0, 4.3 us; the pair 8.2, 20, 4.5).
    constexpr size_t cap = 1u << 20;
    const bool few = a.row_tiles <= 256;
    a.wave_tiles = !few && a.row_bytes * 16 * (pair ? 2 : 1) <= 4096;
    a.waves = few ? 1 : kPackWaves;
    const int runs = (a.nkb + kPackRun - 1) / kPackRun, columns = few ? (runs < 65535 ? runs : 65535) : 1;
    const int share = few ? columns : a.wave_tiles ? 1 : kPackWaves;  // wavefronts of a tile
    a.kb_step = share * kPackRun;
    const size_t groups = a.wave_tiles ? (a.row_tiles + kPackWaves - 1) / kPackWaves : a.row_tiles;
    const dim3 grid((unsigned)(groups < cap ? groups : cap), columns), block(a.waves * kWave);
    a.t_step = (size_t)grid.x * (a.wave_tiles ? kPackWaves : 1);
    auto go = [&](auto vecs) {
        constexpr int V = decltype(vecs)::value;
        if (pair) hipLaunchKernelGGL((pack_kernel<V, 2>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((pack_kernel<V, 1>), grid, block, 0, stream, a);
    };
    if (fmt == 0) go(std::integral_constant<int, 4>{});
    else if (fmt == 1) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

hipError_t launch_pack(int fmt, int E, int N, int K, const void *w, const void *s, void *wp, void *sp,
                       hipStream_t stream)
{
    return pack(fmt, E, N, K, w, s, nullptr, nullptr, wp, sp, nullptr, 0, stream);
}

hipError_t launch_pack_down(int fmt, int E, int N, int K, const void *w, const void *s, void *wp, void *sp,
                            hipStream_t stream)
{
    return pack(fmt, E, N, K, w, s, nullptr, nullptr, wp, sp, nullptr, 1, stream);
}

hipError_t launch_pack_gate_up(int fmt, int E, int N, int K, const void *wg, const void *sg, const void *wu,
                               const void *su, void *wp, void *sgp, void *sup, hipStream_t stream)
{
    return pack(fmt, E, N, K, wg, sg, wu, su, wp, sgp, sup, 0, stream);
}

}  // namespace ecospec
