// The verification pass of small calls (T <= 16 tokens) on gfx950: every
// expert serves at most one 16-token block, unless tokens name it more than once
// (rows padded with zeros do).
//
// These calls are bound by the weight stream and by the latency of its
// launches, so the kernels differ from the general ones (expert_ffn.hip) in
// how a workgroup's wavefronts share an item and in what a launch has to
// build before its first weight load.
//
// Items.  An item is one 16-row tile of W_gate with the same tile of W_up, or
// 32 rows of W_down, over the whole reduction.  Its 128-wide K blocks are
// divided over the workgroup's eight wavefronts (an eighth of the reduction
// each, taken in J rounds of one block; short reductions over fewer, with
// several items side by side: waves_per_item), so an item is one contiguous run
// of memory and every wavefront keeps the same K blocks from item to item.  The
// activations those blocks need (16 tokens x 128 elements each) therefore stay
// in registers, as matrix-core operands, for all items of an expert: no
// activation tiles, and no barrier per step.  The partial sums of an item are
// added through LDS, in wavefront order, by one wavefront (a different one each
// item), behind the item's one barrier.  So a sum over K is up to eight partial
// sums in fp32, where the general kernels add it up in one: single values of y
// differ by a bf16 step, at the same distance from a 64-bit result.  Dealing the
// blocks round-robin instead (a round then reads 32 contiguous KiB) measured the
// same to 2% slower.
//
// Split.  The items of a launch (expert-major) are cut into contiguous ranges
// of whole items, one per workgroup, in closed form from the number of distinct
// experts alone: no cost prefix, no search, no schedule, no sums across
// workgroups and so no fix-up launch.  A range is at most one item longer than
// another; the workgroups still streaming then share the bandwidth of the idle
// ones.  Cutting gate/up items at K blocks where that idle time looked long,
// with the pieces added by the down launch, was slower wherever it applied (the
// launches of one call, without the router, replayed from a graph): Qwen T = 4 on
// 13 experts 83.6 -> 88.6 us, one Qwen expert (96 items on 256 workgroups) 22.8 ->
// 32.9 us.  Cutting down items between their two row tiles gained nothing either
// (GPT-OSS T = 16 on 16 experts 50.8 -> 51.8 us).
//
// H and O rows sit at the routed slots (t * k + j; the shared expert's at
// T * k + t).  A launch needs no grouping: the distinct experts are a bit set
// in LDS and an expert's slots are found with ballots.  An expert of more than
// 16 slots takes part once more for each further 16 (`extra`, built only if one
// of the slots' counts says so).  The routing arrays of the caller (counts,
// union, offsets, perm) are written by one extra workgroup of the combine launch,
// beside the others.
//
// Measured against the general kernels, timed in turn on one box.  Whole calls
// through the Python binding: GPT-OSS T = 1 47.2 -> 27.0 us (with a leaner host
// call), 8 GPT-OSS layers with their routers at T = 4 in one graph 596 -> 437 us,
// Qwen T = 4 (tree routing) 104 -> 84 us, DeepSeek T = 4 on 31 experts 243 -> 232 us,
// T = 16 (tree routing) 357 -> 331 us.  The launches of one call, without router and
// shared expert, replayed from a graph: DeepSeek T = 4 on 31 experts 236.6 -> 214.5
// us, T = 16 on 43 318.6 -> 302.2 us; Qwen T = 16 on 64 379.8 -> 380.1 us; GPT-OSS
// T = 16 on 48 130.9 -> 109.3 us.  At T = 16 each further expert streams at 6.4 (FP8),
// 6.5 (bf16) and 6.7 TB/s (MXFP4; 6.3 before); what is left above the stream is
// about 20 us a call (35 to 40 before).
#include "expert_common.hpp"

namespace ecospec {

constexpr int kSWaves = 8;
constexpr int kSThreads = kSWaves * kWave;
constexpr int kSmallSlots = kSmallT * 64;  // routed slots: k <= 64

// A divisor known before the launch: x / d for x < 2^31 as a multiplication (the 31-bit case of the
// round-up method: m = ceil(2^(31 + s) / d) with s = ceil(log2 d) fits 32 bits and is exact).
struct Divisor {
    uint32_t d, m, s;
    __device__ __forceinline__ uint32_t operator()(uint32_t x) const { return (uint32_t)(((uint64_t)x * m) >> (31 + s)); }
};

static Divisor divisor(uint32_t d)
{
    uint32_t s = 0;
    while ((1ull << s) < d) ++s;
    return Divisor{d, (uint32_t)((((uint64_t)1 << (31 + s)) + d - 1) / d), s};
}

// Where one kind of expert's weights lie (routed, or the shared one): tile 0 and tile 1 of item 0.
struct SmallWeights {
    const uint8_t *w0, *w1, *s0, *s1;
    uint32_t expert;            // bytes from one expert's matrix (pair) to the next
    uint32_t range0, range1;    // bytes of an expert that are readable from w0 and w1 on
    uint32_t kstride, tstride;  // bytes from one K block, and one item, to the next
};

struct SmallParams {
    SmallWeights wts[2];   // the routed experts', the shared expert's
    const int32_t *topk_idx;
    const void *in;        // x or H
    void *out;             // H or O
    const float *b_gate, *b_up;
    int T, k, S, E, U_extra;  // U_extra: 1 with a shared expert
    int K, nblocks, ldo;      // reduction length, its 128-wide blocks, columns of a row of `out`
    uint32_t sc_bytes, sstride;  // bytes of an expert's scales; MXFP4: of one item's
    Divisor dG, dtiles, dk;   // workgroups, items per expert, top-k
    int act;
    float alpha, limit;
};

// Weights of one round of a wavefront: one 16 x 128 block of each of its two tiles.
template <int FMT> struct SmallSlot {
    u32x4 v[2][Fmt<FMT>::kVecs];
    uint32_t sc[2];  // FP8: the block scales' bits; MXFP4: the lane's e8m0 codes of a quad of blocks
};

// Prefetch ring: D rounds in flight per wavefront.  An item is J rounds, padded to JU so that the loop (P items
// unrolled) is a whole number of turns of the ring; J blocks of activations (16 registers each) and D slots (FP8 16
// registers, bf16 32, MXFP4 10) share the 256 registers of a wavefront.  Up to two rounds an item, D is what keeps P
// at one or a few: each unrolled item is a copy of the epilogue, and the copies cost more than the depth brings (32
// experts, T = 4: 128 x 4096 FP8 4 -> 2 rounds 19.8 -> 17.7 us, MXFP4 6 -> 3 19.3 -> 17.7; 2048 x 2048 MXFP4 6 -> 4 47.4 ->
// 45.8).  FP8 keeps four where eight wavefronts share 9 to 16 blocks: with nine, most of them have one block, so that
// two rounds hold one live one (128 experts of 1152 x 1152, T = 16: 90.8 us with four, 94.8 with two; with all 16 blocks
// two are 2% faster).  Beyond that the depth matters little, so these are J itself or a divisor where the
// registers hold it: FP8 with two rounds throughout is 0.6 and 1.0% slower at J = 3 and 4, 1.1 and 0.6% faster at 5 and
// 6; MXFP4 with three or four is 1.4% slower, 1.2% faster, 3.0% and 0.4% slower at J = 3 to 6; bf16 with two instead of three
// is within 0.2% at J = 5 and 6 and 1.3% faster at 3, with three instead of two 3.8% faster at 4 (4096 x 4096) and 2% slower
// for Qwen's J = 4 and 2.  J = 7 padded to eight rounds and not padded (P = 2) are the same (DeepSeek T = 4 213.8, 213.9 us).
template <int FMT, bool DOWN, int J, int KW> struct Ring {
    static constexpr int D = FMT == FMT_FP8    ? (J <= 2 ? (KW < kSWaves ? 2 : 4) : J >= 7 || (DOWN && J == 6) ? 2 : J == 6 ? 3 : J)
                           : FMT == FMT_BF16   ? (J == 3 || J == 5 || J == 6 ? 3 : 2)
                                               : (J == 1 ? 3 : J == 3 ? 6 : J == 4 ? 8 : J == 5 || J == 6 ? J : 4);
    static constexpr int JU = J >= D ? (J + D - 1) / D * D : J;
    static constexpr int P = JU >= D ? 1 : D / JU;
    static_assert((P * JU) % D == 0 && JU >= J, "whole turns of the ring");
};

// KW: wavefronts that share an item; the workgroup takes kSWaves / KW items at a time (a turn).
template <int FMT, bool DOWN, int J, int KW>
__global__ __launch_bounds__(kSThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void expert_small_kernel(SmallParams P)
{
    constexpr int NC = kSWaves / KW;
    constexpr int NV = Fmt<FMT>::kVecs;
    constexpr uint32_t BLK = 1024u * NV;
    using R = Ring<FMT, DOWN, J, KW>;
    constexpr int D = R::D, JU = R::JU, PU = R::P;
    __shared__ uint32_t emask[32];                // distinct routed experts (E <= 1024)
    __shared__ int cnt[1024];                     // slots of each expert
    __shared__ int extra[kSmallSlots / kSmallT];  // expert | first slot << 16 of each block of slots past an expert's first
    __shared__ int n_extra;                       // their number; -1: to be counted
    __shared__ int sidx[kSmallSlots];             // expert of each routed slot
    __shared__ int slots[kSWaves][kSmallT];       // slots of the current expert (one copy per wavefront)
    __shared__ f32x4 red[2][kSWaves][2][kWave];   // an item's partial sums, double-buffered
    const uint32_t G = P.dG.d;
    // Ranges XCD-major: the workgroups sharing an L2 work on neighbouring items.
    const uint32_t w = G % 8 == 0 ? (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8 : blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), col = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int sub = NC == 1 ? 0 : wave / KW, part = NC == 1 ? wave : wave % KW;
    const int S = P.S;

    // Distinct experts.
    if (tid < 32) emask[tid] = 0u;
    cnt[tid] = cnt[tid + kSThreads] = 0;
    if (tid == 0) n_extra = 0;
    const int e0 = tid < S ? P.topk_idx[tid] : -1, e1 = tid + kSThreads < S ? P.topk_idx[tid + kSThreads] : -1;
    fetch_args(P);  // in the shadow of the slots' load
    __syncthreads();
    auto enter = [&](int slot, int e) {
        if (slot < S) sidx[slot] = e;
        if ((unsigned)e < (unsigned)P.E) {
            atomicOr(&emask[e >> 5], 1u << (e & 31));
            if (S > kSmallT && atomicAdd(&cnt[e], 1) >= kSmallT) n_extra = -1;
        }
    };
    enter(tid, e0);
    if (S > kSThreads) enter(tid + kSThreads, e1);
    __syncthreads();
    if (n_extra < 0) {
        __syncthreads();
        if (wave == 0) {
            int n = 0;
            for (int e = lane; e < 1024; e += kWave) {
                const int more = (max(cnt[e], 1) - 1) / kSmallT, incl = wave_inclusive_sum(more);
                for (int b = 0; b < more; ++b) extra[n + incl - more + b] = e | (kSmallT * (b + 1)) << 16;
                n += __builtin_amdgcn_readlane(incl, 63);
            }
            if (lane == 0) n_extra = n;
        }
        __syncthreads();
    }
    const uint32_t mword = lane < 32 ? emask[lane] : 0u;
    const int mcount = __popc(mword), mincl = wave_inclusive_sum(mcount);
    const int U = __builtin_amdgcn_readlane(mincl, 63);
    const int n_first = U + P.U_extra;
    const uint32_t n_exp = (uint32_t)(n_first + __builtin_amdgcn_readfirstlane(n_extra));
    // Id of the u-th expert: the distinct ones, the shared expert (-1), then those of `extra` (wave-uniform).
    auto expert_of = [&](int u) -> int {
        if (u >= n_first) return __builtin_amdgcn_readfirstlane(extra[u - n_first]) & 0xffff;
        if (u >= U) return -1;
        const int wl = __builtin_ctzll(__ballot(mincl > u && mincl - mcount <= u));
        const uint32_t word = __builtin_amdgcn_readlane(mword, wl);
        const int r = u - __builtin_amdgcn_readlane(mincl - mcount, wl);
        const uint32_t below = (1u << (lane & 31)) - 1u;
        const uint64_t hit = __ballot(lane < 32 && ((word >> lane) & 1u) && __popc(word & below) == r);
        return 32 * wl + (int)__builtin_ctzll(hit);
    };

    const uint32_t items = n_exp * P.dtiles.d;  // items * (G + 1) < 2^31
    const uint32_t x0 = P.dG(items * w), x1 = P.dG(items * (w + 1));
    if (x0 >= x1) return;
    const int n = (int)(x1 - x0);  // items of the range
    const int nkb = P.nblocks, tiles = (int)P.dtiles.d;
    const int kb0 = nkb * part / KW, kcount = nkb * (part + 1) / KW - kb0;  // this wavefront's K blocks
    const int mine_n = NC == 1 ? n : sub < n ? (n - sub + NC - 1) / NC : 0;  // its items: x0 + sub, x0 + sub + NC, ...
    const uint32_t xs = NC == 1 ? x0 : x0 + (sub < n ? sub : 0);
    const int u0 = (int)P.dtiles(xs), it0 = (int)xs - u0 * tiles;

    // On to the wavefront's next item, tile t of expert u; `enter` is called if that is another expert (and there
    // are more items).
    auto next_item = [&](int &t, int &u, bool more, auto &&enter) __attribute__((always_inline)) {
        if constexpr (NC == 1) {
            if (++t == tiles) {
                t = 0;
                if (more) enter(++u);
            }
        } else {
            t += NC;
            if (t < tiles) return;
            do {
                t -= tiles;
                ++u;
            } while (t >= tiles);
            if (more) enter(u);
        }
    };

    // Load cursor: the item whose weights are being issued.  Offsets are scalar: a load's address is its
    // descriptor's base + wj + the lane's 16 bytes.  A dead load (past the range, or a block another
    // wavefront has) moves every lane out of the descriptor's range and reads zeros; its scalar offset is 0,
    // since the range check compares with the range less that offset.
    rsrc_t ra0, ra1, rs0, rs1;
    uint32_t kstride, tstride;
    auto set_expert = [&](int u) {
        const int e = expert_of(u);
        const SmallWeights &q = P.wts[e < 0 ? 1 : 0];
        const size_t ee = e < 0 ? 0 : (size_t)e;
        ra0 = make_rsrc(q.w0 + ee * q.expert, q.range0);
        ra1 = make_rsrc(q.w1 + ee * q.expert, q.range1);
        kstride = q.kstride;
        tstride = q.tstride;
        if constexpr (FMT != FMT_BF16) {
            rs0 = make_rsrc(q.s0 + ee * P.sc_bytes, P.sc_bytes);
            rs1 = make_rsrc(q.s1 + ee * P.sc_bytes, P.sc_bytes);
        }
    };
    set_expert(u0);
    int ci = 0, ct = it0, cu = u0, jhi = NC == 1 || mine_n > 0 ? kcount : 0;
    uint32_t wj = (uint32_t)ct * tstride + (uint32_t)kb0 * kstride;
    auto advance = [&]() {
        ++ci;
        next_item(ct, cu, ci < mine_n, set_expert);
        jhi = ci < mine_n ? kcount : 0;
        wj = (uint32_t)ct * tstride + (uint32_t)kb0 * kstride;
    };

    SmallSlot<FMT> ring[D];
    const uint32_t lane16 = (uint32_t)lane * 16u, lane4 = (uint32_t)lane * 4u;
    auto issue = [&](int slot, int j) {
        int h = jhi;
        asm volatile("" : "+s"(h));  // not an invariant to be kept in vector registers for every j
        const bool live = j < h;
        const uint32_t dead = live ? 0u : kOff, vo = lane16 | dead;
        const int wo = live ? (int)wj : 0;
#pragma unroll
        for (int i = 0; i < NV; ++i)
            ring[slot].v[0][i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ra0, (int)(vo + 1024u * i), wo, kAuxNT));
#pragma unroll
        for (int i = 0; i < NV; ++i)
            ring[slot].v[1][i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ra1, (int)(vo + 1024u * i), wo, kAuxNT));
        wj += kstride;
        if constexpr (FMT == FMT_FP8) {  // 128 x 128 block scales: an item's rows lie in one row block
            const int so = live ? ((ct / (DOWN ? 4 : 8)) * nkb + kb0 + j) * 4 : 0;
            ring[slot].sc[0] = __builtin_amdgcn_raw_buffer_load_b32(rs0, (int)dead, so, 0);
            ring[slot].sc[1] = DOWN ? ring[slot].sc[0] : __builtin_amdgcn_raw_buffer_load_b32(rs1, (int)dead, so, 0);
        } else if constexpr (FMT == FMT_MXFP4) {
            const int so = live ? ct * (int)P.sstride + ((kb0 + j) >> 2) * 256 : 0;
            ring[slot].sc[0] = __builtin_amdgcn_raw_buffer_load_b32(rs0, (int)(lane4 | dead), so, 0);
            ring[slot].sc[1] = __builtin_amdgcn_raw_buffer_load_b32(rs1, (int)(lane4 | dead), so, 0);
        }
    };

    // The current expert's slots and the wavefront's activation blocks (B operands): lane (col, grp) holds
    // token col's elements kb * 128 + 32 grp .. + 31 of each block.
    int myslot = -1, ce = -1;
    bf16x8 bx[J][4];
    const uint32_t brow = (uint32_t)P.K * 2u;
    const rsrc_t rb = make_rsrc(P.in, (uint32_t)(DOWN ? S + P.U_extra * P.T : P.T) * brow);
    auto load_b = [&](int u) {
        ce = expert_of(u);
        if (ce < 0) {
            myslot = col < P.T ? S + col : -1;
        } else {
            const int skip = u >= n_first ? __builtin_amdgcn_readfirstlane(extra[u - n_first]) >> 16 : 0;
            int cnt = -skip;
            for (int base = 0; base < S; base += kWave) {
                const bool hit = base + lane < S && sidx[base + lane] == ce;
                const uint64_t m = __ballot(hit);
                const int r = cnt + __popcll(m & ((1ull << lane) - 1ull));
                if (hit && (unsigned)r < (unsigned)kSmallT) slots[wave][r] = base + lane;
                cnt += __popcll(m);
            }
            __builtin_amdgcn_wave_barrier();  // the same wavefront's LDS accesses stay in order
            myslot = col < cnt ? slots[wave][col] : -1;
        }
        const uint32_t row = (uint32_t)(DOWN ? myslot : ce < 0 ? myslot - S : (int)P.dk((uint32_t)myslot & 0x7fffffffu));
        const uint32_t off = myslot >= 0 ? row * brow + 64u * grp : kOff;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int k0 = (kb0 + j) * kMacroK;  // K % 32 == 0: a lane's chunk is all in or all out
            const uint32_t vo = j < kcount && k0 + 32 * grp < P.K ? off : kOff;
            const int so = j < kcount ? 2 * k0 : 0;
#pragma unroll
            for (int s = 0; s < 4; ++s)
                bx[j][s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rb, (int)(vo + 16u * s), so, 0));
        }
    };

    // Pipeline prologue: the first item's weights, the activations, then the rest of the ring.
    int bu = u0, bt = it0;  // expert and tile being contracted
#pragma unroll
    for (int q = 0; q < D - 1; ++q) {
        if (q > 0 && q % JU == 0) advance();
        issue(q, q % JU);
        if (q == (J < D - 1 ? J : D - 1) - 1 && (NC == 1 || mine_n > 0)) load_b(bu);
    }
    const bool biased = !DOWN && (P.b_gate != nullptr || P.b_up != nullptr);
    const int turns = (n + NC - 1) / NC;
    for (int i0 = 0; i0 < turns; i0 += PU) {
#pragma unroll
        for (int p = 0; p < PU; ++p) {
            const int i = i0 + p;
            const bool mine = part == (i & (KW - 1));  // this wavefront finishes the item
            f32x4 gb = f32x4{0.f, 0.f, 0.f, 0.f}, ub = gb;
            if (biased && mine && i < mine_n && ce >= 0) {
                const size_t o = (size_t)ce * P.ldo + 16 * bt + 4 * grp;
                if (P.b_gate) gb = *reinterpret_cast<const f32x4 *>(P.b_gate + o);
                if (P.b_up) ub = *reinterpret_cast<const f32x4 *>(P.b_up + o);
            }
            f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
            const int live_rounds = i < mine_n ? kcount : 0;
#pragma unroll
            for (int j = 0; j < JU; ++j) {
                const int q = p * JU + j + D - 1;  // the round whose loads go out now
                if (q % JU == 0) advance();
                issue(q % D, q % JU);
                // A branch per round, on a value opaque to the compiler: without it, it interleaves the rounds'
                // decoding and spills (FP8, J = 7: 18 registers; DeepSeek T = 4 227 -> 248 us).
                int jlive = live_rounds;
                asm volatile("" : "+s"(jlive));
                if (j < jlive) {
                    const SmallSlot<FMT> &sl = ring[(p * JU + j) % D];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const float sc = FMT == FMT_MXFP4 ? e8m0_scale_operand(sl.sc[t] >> (8 * ((kb0 + j) & 3))) : 1.f;
                        f32x4 c = FMT == FMT_FP8 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[t];
#pragma unroll
                        for (int s = 0; s < 4; ++s)
                            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(decode8<FMT>(sl.v[t], s, sc), bx[j < J ? j : 0][s], c,
                                                                        0, 0, 0);
                        if constexpr (FMT == FMT_FP8) {
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                acc[t][r] = __builtin_fmaf(__uint_as_float(sl.sc[t]), c[r], acc[t][r]);
                        } else {
                            acc[t] = c;
                        }
                    }
                }
            }
            if (i < turns) {
                const int buf = i & 1;
                if constexpr (KW > 1) {
                    red[buf][wave][0][lane] = acc[0];
                    red[buf][wave][1][lane] = acc[1];
                    // LDS only: the weight loads in flight stay in flight.  A turn's sums are read before the
                    // next turn's barrier and overwritten after it.
                    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                }
                if (mine && (NC == 1 || i < mine_n)) {
                    f32x4 r0 = acc[0], r1 = acc[1];
                    if constexpr (KW > 1) {
                        r0 = red[buf][sub * KW][0][lane];
                        r1 = red[buf][sub * KW][1][lane];
#pragma unroll
                        for (int v = 1; v < KW; ++v) {
                            r0 += red[buf][sub * KW + v][0][lane];
                            r1 += red[buf][sub * KW + v][1][lane];
                        }
                    }
                    if (DOWN) {
                        if (myslot >= 0) {
                            float *dst = static_cast<float *>(P.out) + (size_t)myslot * P.ldo + 32 * bt + 4 * grp;
                            *reinterpret_cast<f32x4 *>(dst) = r0;
                            *reinterpret_cast<f32x4 *>(dst + 16) = r1;
                        }
                    } else if (myslot >= 0) {
                        r0 += gb;
                        r1 += ub;
                        float h[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) h[r] = activate(P.act, P.alpha, P.limit, r0[r], r1[r]);
                        *reinterpret_cast<u32x2 *>(static_cast<uint16_t *>(P.out) + (size_t)myslot * P.ldo + 16 * bt + 4 * grp) =
                            u32x2{pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3])};
                    }
                }
                next_item(bt, bu, i + 1 < mine_n, load_b);
            }
        }
    }
}

// The union and grouping of the routed slots (Eq. 1) into the caller's routing arrays, as moe_expert_union
// computes them, by one 256-thread workgroup (S <= 1024 slots, E <= 1024 experts).
__device__ __forceinline__ void small_union(const VerifyArgs &a)
{
    __shared__ int cnt[1024], start[1024], wave_tot[2 * 256 / kWave];
    const int tid = threadIdx.x, wave = tid / kWave, S = a.T * a.k, E = a.E;
    int nbits = 0;
    while ((1 << nbits) < E) ++nbits;
    for (int e = tid; e < E; e += 256) cnt[e] = 0;
    __syncthreads();
    for (int s = tid; s < S; s += 256) {
        const int e = a.topk_idx[s];
        if ((unsigned)e < (unsigned)E) atomicAdd(&cnt[e], 1);
    }
    __syncthreads();
    int c[4], used = 0, sum = 0;  // experts 4 tid .. 4 tid + 3
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c[i] = 4 * tid + i < E ? cnt[4 * tid + i] : 0;
        used += c[i] > 0;
        sum += c[i];
    }
    int pos, off, U, placed;
    block_exclusive_scan2(used, sum, wave_tot, pos, off, U, placed);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = 4 * tid + i;
        if (e < E) {
            a.counts[e] = c[i];
            start[e] = off;
            if (c[i] > 0) {
                a.union_ids[pos] = e;
                a.offsets[pos] = off;
                ++pos;
                off += c[i];
            }
        }
    }
    for (int u = U + tid; u <= E; u += 256) {
        if (u < E) a.union_ids[u] = -1;
        a.offsets[u] = placed;
    }
    if (tid == 0) *a.n_unique = U;
    __syncthreads();
    // Placement, a wavefront at a time: first position of the expert + its slots before + rank.
    for (int base = 0; base < S; base += 256) {
        const int s = base + tid, e = s < S ? a.topk_idx[s] : -1;
        const bool ok = (unsigned)e < (unsigned)E;
        int rank, count;
        bool top;
        wave_match(e, ok, nbits, rank, top, count);
        for (int v = 0; v < 256 / kWave && base + v * kWave < S; ++v) {
            if (v == wave && ok) {
                const int p = start[e];
                a.perm[p + rank] = s;
                if (top) start[e] = p + count;
            }
            __syncthreads();
        }
    }
}

// y[t] = sum_j w[t][j] * (O[slot] + b_down[expert]) (+ shared) -> bf16, in the order j = 0 .. k-1, then the
// shared expert; 4 columns per thread.  Every row of O is whole, so all loads of eight slots go out in one round
// trip.  The last workgroup writes the routing arrays instead.
__global__ __launch_bounds__(256) void combine_small_kernel(VerifyArgs a)
{
    fetch_args(a);
    if (blockIdx.x == gridDim.x - 1) {
        small_union(a);
        return;
    }
    constexpr int CH = 8;
    const int per_row = a.d / 4;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= a.T * per_row) return;
    const int t = i / per_row, c = (i - t * per_row) * 4;
    const int S = a.T * a.k;
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f}, vsh = s;
    if (a.sh_gate) vsh = *reinterpret_cast<const f32x4 *>(a.o + (size_t)(S + t) * a.d + c);
    for (int j0 = 0; j0 < a.k; j0 += CH) {
        int ej[CH];
        float wj[CH];
        f32x4 vj[CH];
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const int slot = t * a.k + min(j0 + q, a.k - 1);
            ej[q] = j0 + q < a.k ? a.topk_idx[slot] : -1;
            wj[q] = a.topk_w[slot];
            vj[q] = *reinterpret_cast<const f32x4 *>(a.o + (size_t)slot * a.d + c);
        }
        // A slot whose expert lies outside [0, E) has no row of O: it adds nothing.
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const bool ok = (unsigned)ej[q] < (unsigned)a.E;
            if (a.b_down && ok) vj[q] += *reinterpret_cast<const f32x4 *>(a.b_down + (size_t)ej[q] * a.d + c);
            if (ok) s += wj[q] * vj[q];
        }
    }
    if (a.sh_gate) s += vsh;
    *reinterpret_cast<u32x2 *>(a.y + (size_t)t * a.d + c) = u32x2{pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3])};
}

// ----------------------------------------------------------------------------- host side

// Wavefronts that share an item: eight, or, for reductions of up to eight blocks, the fewest that leave each at most
// two rounds (bf16) or three (FP8, MXFP4, whose rounds are half and a quarter as long).  With eight throughout, such
// reductions left wavefronts without a block and paid the item's barrier for a few KiB, at least 0.7 us per item: 128
// experts of 128 x 8192 (T = 16) took 235 us in bf16, 204 in FP8 and 191 in MXFP4 (the general kernels 141, 100 and 106),
// now 132, 70 and 52; 640 x 2176 in MXFP4 84 (general 83), now 57; 2048 x 768 in MXFP4 74 (general 71), now 63.  Three
// rounds against two: 2048 x 768 in FP8 at T = 1 16.6 us against 17.5, in bf16 21.8 against 20.7.
static int waves_per_item(int fmt, int nblocks)
{
    if (nblocks > 8) return kSWaves;
    int kw = 1;
    while ((nblocks + kw - 1) / kw > (fmt == FMT_BF16 ? 2 : 3)) kw *= 2;
    return kw;
}

template <int FMT, bool DOWN>
static hipError_t launch_projection(const SmallParams &p, int workers, hipStream_t stream)
{
    const dim3 grid(workers), block(kSThreads);
    const int kw = waves_per_item(FMT, p.nblocks), rounds = (p.nblocks + kw - 1) / kw;
    switch (kw * 16 + rounds) {
#define SMALL_CASE(KW, J)                                                                              \
    case KW * 16 + J:                                                                                  \
        if constexpr (KW == kSWaves || J <= 2 || FMT != FMT_BF16)                                      \
            hipLaunchKernelGGL((expert_small_kernel<FMT, DOWN, J, KW>), grid, block, 0, stream, p);    \
        break;
        SMALL_CASE(1, 1) SMALL_CASE(1, 2) SMALL_CASE(1, 3) SMALL_CASE(2, 2) SMALL_CASE(2, 3) SMALL_CASE(4, 2)
        SMALL_CASE(8, 2) SMALL_CASE(8, 3) SMALL_CASE(8, 4) SMALL_CASE(8, 5) SMALL_CASE(8, 6) SMALL_CASE(8, 7) SMALL_CASE(8, 8)
#undef SMALL_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

bool small_verify(const VerifyArgs &a, int workers)
{
    const int nu = (a.d + kMacroK - 1) / kMacroK, nd = (a.d_ff + kMacroK - 1) / kMacroK;
    if (a.T > kSmallT || a.act_fmt != 0 || nu > 8 * kSWaves || nd > 8 * kSWaves) return false;
    // The split's arithmetic is 32-bit.
    const uint64_t n_exp = (uint64_t)(a.E < a.T * a.k ? a.E : a.T * a.k) + 1 + a.T * a.k / kSmallT;
    const uint64_t items = n_exp * (uint64_t)(a.d_ff / 16 > a.d / 32 ? a.d_ff / 16 : a.d / 32);
    return items * ((uint64_t)workers + 1) < (1ull << 31);
}

// The weights of the routed or of the shared expert for one launch: `w` (and, unpaired gate/up, `w2`).
template <int FMT>
static SmallWeights small_weights(bool down, bool pair, const uint8_t *w, const uint8_t *w2, const void *s, const void *s2, int N,
                                  int K)
{
    constexpr uint32_t BLK = 1024u * Fmt<FMT>::kVecs;
    const uint32_t mat = (uint32_t)packed_matrix_bytes(FMT, N, K), nkb = (uint32_t)(K + kMacroK - 1) / kMacroK;
    SmallWeights q{};
    if (!w) return q;
    q.s0 = static_cast<const uint8_t *>(s);
    q.s1 = static_cast<const uint8_t *>(s2);
    q.w0 = w;
    q.kstride = pair ? 2 * BLK : BLK;
    q.tstride = nkb * BLK * (down || pair ? 2 : 1);
    const uint32_t toff = pair ? BLK : down ? nkb * BLK : 0;  // tile 1's first block, from tile 0's
    q.w1 = (!down && !pair ? w2 : w) + toff;
    q.expert = q.range0 = mat * (!down && pair ? 2u : 1u);
    q.range1 = q.range0 - toff;
    return q;
}

template <int FMT>
static hipError_t launch_small_fmt(const VerifyArgs &args, uint8_t *ws_base, const VerifyWorkspace &ws, hipStream_t stream,
                                   hipEvent_t const *events)
{
    auto mark = [&](int i) { return events && events[i] ? hipEventRecord(events[i], stream) : hipSuccess; };
    VerifyArgs a = args;
    a.h = reinterpret_cast<uint16_t *>(ws_base + ws.h_offset);
    a.o = reinterpret_cast<float *>(ws_base + ws.o_offset);
    SmallParams p{};
    p.topk_idx = a.topk_idx;
    p.b_gate = a.b_gate;
    p.b_up = a.b_up;
    p.T = a.T;
    p.k = a.k;
    p.S = a.T * a.k;
    p.E = a.E;
    p.U_extra = a.sh_gate ? 1 : 0;
    p.dG = divisor((uint32_t)ws.workers);
    p.dk = divisor((uint32_t)a.k);
    p.act = a.act;
    p.alpha = a.alpha;
    p.limit = a.limit;

    auto geometry = [&](bool down, int N, int K) {
        p.K = K;
        p.ldo = N;
        p.nblocks = (K + kMacroK - 1) / kMacroK;
        p.dtiles = divisor((uint32_t)(down ? N / 32 : N / 16));
        p.sc_bytes = (uint32_t)packed_scale_bytes(FMT, N, K);
        p.sstride = (down ? 2u : 1u) * (uint32_t)((p.nblocks + 3) / 4) * 256u;
    };
    geometry(false, a.d_ff, a.d);
    p.wts[0] = small_weights<FMT>(false, a.gu_pair, a.w_gate, a.w_up, a.s_gate, a.s_up, a.d_ff, a.d);
    p.wts[1] = small_weights<FMT>(false, a.sh_gu_pair, a.sh_gate, a.sh_up, a.sh_s_gate, a.sh_s_up, a.d_ff, a.d);
    p.in = a.x;
    p.out = a.h;
    hipError_t err;
    if ((err = mark(0)) != hipSuccess) return err;
    if ((err = launch_projection<FMT, false>(p, ws.workers, stream)) != hipSuccess) return err;
    if ((err = mark(1)) != hipSuccess) return err;

    geometry(true, a.d, a.d_ff);
    // MXFP4 scales of the second row tile of an item lie one row tile further.
    const size_t s1 = FMT == FMT_MXFP4 ? p.sstride / 2 : 0;
    auto after = [&](const void *s) { return static_cast<const uint8_t *>(s) + s1; };
    p.wts[0] = small_weights<FMT>(true, a.down_pair, a.w_down, nullptr, a.s_down, after(a.s_down), a.d, a.d_ff);
    p.wts[1] = small_weights<FMT>(true, a.down_pair, a.sh_down, nullptr, a.sh_s_down, after(a.sh_s_down), a.d, a.d_ff);
    p.in = a.h;
    p.out = a.o;
    if ((err = mark(2)) != hipSuccess) return err;
    if ((err = launch_projection<FMT, true>(p, ws.workers, stream)) != hipSuccess) return err;
    if ((err = mark(3)) != hipSuccess) return err;
    hipLaunchKernelGGL(combine_small_kernel, dim3((a.T * (a.d / 4) + 255) / 256 + 1), dim3(256), 0, stream, a);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    return mark(4);
}

hipError_t launch_small_verify(const VerifyArgs &a, void *workspace, const VerifyWorkspace &ws, hipStream_t stream,
                               hipEvent_t const *events)
{
    uint8_t *base = static_cast<uint8_t *>(workspace);
    switch (a.fmt) {
    case FMT_BF16: return launch_small_fmt<FMT_BF16>(a, base, ws, stream, events);
    case FMT_FP8: return launch_small_fmt<FMT_FP8>(a, base, ws, stream, events);
    case FMT_MXFP4: return launch_small_fmt<FMT_MXFP4>(a, base, ws, stream, events);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ecospec
