// The verification pass of small calls (T <= 16 tokens) on gfx950: every
// expert serves at most one 16-token block.
//
// These calls are bound by the weight stream and by the latency of its
// launches, so the kernels differ from the general ones (expert_ffn.hip) in
// how a workgroup's wavefronts share an item and in what a launch has to
// build before its first weight load.
//
// Items.  An item is one 16-row tile of W_gate with the same tile of W_up, or
// 32 rows of W_down, over the whole reduction.  Its 128-wide K blocks are
// divided over the workgroup's eight wavefronts (an eighth of the reduction
// each, taken in J rounds of one block), so an item is one contiguous run of
// memory and every wavefront keeps the same K blocks from item to item.  The
// activations those blocks need (16 tokens x 128 elements each) therefore stay
// in registers, as matrix-core operands, for all items of an expert: no
// activation tiles, and no barrier per step.  The eight partial sums of an
// item are added through LDS, in wavefront order, by one wavefront (a
// different one each item), behind the item's one barrier.  Dealing the blocks
// round-robin instead (a round then reads 32 contiguous KiB) measured the same
// to 2% slower; rings of half or twice the depth are no faster.
//
// Split.  The items of a launch (expert-major) are cut into equal contiguous
// ranges, one per workgroup, in closed form from the number of distinct
// experts alone: no cost prefix, no search, no schedule.  Ranges normally hold
// whole items.  Where whole items would leave the workgroups idle for long
// (few, large items) the gate/up ranges are cut at rounds instead; the pieces
// of a cut item stay in the workspace as fp32 sums and the down launch adds
// them, in workgroup order, as it loads its activations, finding them with the
// same closed form.  There is no fix-up launch.
//
// H and O rows sit at the routed slots (t * k + j; the shared expert's at
// T * k + t).  A launch needs no grouping: the distinct experts are a bit set
// in LDS and an expert's slots are found with ballots.  The routing arrays of
// the caller (counts, union, offsets, perm) are written by one extra workgroup
// of the combine launch, beside the others.
//
// Measured against the general kernels (whole pass, same box): GPT-OSS layer
// T = 1 47.1 -> 33.7 us, T = 4 (8-layer graph, with its router) 594 -> 466 us;
// Qwen layer T = 4, 13 experts 105.6 -> 91.3 us; DeepSeek layer T = 4,
// 31 experts 236.9 -> 231.5 us, T = 16, 37 experts 324 -> 309 us.  At T = 16 each
// further expert streams at 6.4 (FP8), 6.5 (bf16) and 6.7 TB/s (MXFP4; 6.3
// before); what is left above the stream is 22 us a pass (35 to 40 before).
#include "expert_common.hpp"
#include "split.hpp"

namespace ecospec {

constexpr int kSWaves = 8;
constexpr int kSThreads = kSWaves * kWave;
constexpr int kSmallSlots = kSmallT * 64;  // routed slots: k <= 64
constexpr int kPieceFloats = 2 * kWave * 4;  // partial sums of one piece of a cut item (gate and up tile)

struct SmallParams {
    VerifyArgs a;
    int N, K;              // rows and reduction length of one streamed matrix
    int nblocks;           // 128-wide K blocks
    int tiles;             // items per expert
    uint32_t mat_bytes, sc_bytes;
    int workers;
    float *pieces;         // [workers][2][kPieceFloats]
    int gu_tiles, gu_rounds;  // the gate/up launch's items per expert and rounds per item
    uint32_t gu_bytes;        // and bytes per item
};

// Weights of one round of a wavefront: one 16 x 128 block of each of its two tiles.
template <int FMT> struct SmallSlot {
    u32x4 v[2][Fmt<FMT>::kVecs];
    uint32_t sc[2];  // FP8: the block scales' bits; MXFP4: the lane's e8m0 codes of a quad of blocks
};

// Prefetch ring: D rounds in flight per wavefront.  An item is J rounds, padded to JU so that the loop
// (P items unrolled) is a whole number of turns of the ring; J blocks of activations (16 registers each)
// and D slots share the 256 registers of a wavefront (the down kernels need a few more than gate/up).
template <int FMT, bool DOWN, int J> struct Ring {
    static constexpr int D = FMT == FMT_FP8    ? (DOWN && J >= 6 ? 2 : J == 3 || J == 5 || J == 6 ? J : 4)
                           : FMT == FMT_BF16   ? (J == 1 || J == 3 || J == 5 || J == 6 ? 3 : J >= 7 ? 2 : 4)
                                               : (J <= 3 ? 6 : J == 4 ? 8 : J <= 6 ? J : 4);
    static constexpr int JU = J >= D ? (J + D - 1) / D * D : J;
    static constexpr int P = JU >= D ? 1 : D / JU;
    static_assert((P * JU) % D == 0 && JU >= J, "whole turns of the ring");
};

template <int FMT, bool DOWN, int J>
__global__ __launch_bounds__(kSThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void expert_small_kernel(SmallParams P)
{
    constexpr int NV = Fmt<FMT>::kVecs;
    constexpr uint32_t BLK = 1024u * NV;
    using R = Ring<FMT, DOWN, J>;
    constexpr int D = R::D, JU = R::JU, PU = R::P;
    __shared__ uint32_t emask[32];                // distinct routed experts (E <= 1024)
    __shared__ int sidx[kSmallSlots];             // expert of each routed slot
    __shared__ int slots[kSWaves][kSmallT];       // slots of the current expert (one copy per wavefront)
    __shared__ f32x4 red[2][kSWaves][2][kWave];   // an item's partial sums, double-buffered
    const VerifyArgs &a = P.a;
    const uint32_t G = (uint32_t)P.workers;
    // Ranges XCD-major: the workgroups sharing an L2 work on neighbouring items.
    const uint32_t w = G % 8 == 0 ? (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8 : blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), col = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int S = a.T * a.k;

    // Distinct experts.
    if (tid < 32) emask[tid] = 0u;
    int e0 = tid < S ? a.topk_idx[tid] : -1, e1 = tid + kSThreads < S ? a.topk_idx[tid + kSThreads] : -1;
    __syncthreads();
    if (tid < S) sidx[tid] = e0;
    if (tid + kSThreads < S) sidx[tid + kSThreads] = e1;
    if ((unsigned)e0 < (unsigned)a.E) atomicOr(&emask[e0 >> 5], 1u << (e0 & 31));
    if ((unsigned)e1 < (unsigned)a.E) atomicOr(&emask[e1 >> 5], 1u << (e1 & 31));
    __syncthreads();
    const uint32_t mword = lane < 32 ? emask[lane] : 0u;
    const int mcount = __popc(mword), mincl = wave_inclusive_sum(mcount);
    const int U = __builtin_amdgcn_readlane(mincl, 63);
    const uint32_t n_exp = (uint32_t)(U + (a.sh_gate ? 1 : 0));
    // Id of the u-th distinct expert (wave-uniform; -1: the shared expert).
    auto expert_of = [&](int u) -> int {
        if (u >= U) return -1;
        const int wl = __builtin_ctzll(__ballot(mincl > u && mincl - mcount <= u));
        const uint32_t word = __builtin_amdgcn_readlane(mword, wl);
        const int r = u - __builtin_amdgcn_readlane(mincl - mcount, wl);
        const uint32_t below = (1u << (lane & 31)) - 1u;
        const uint64_t hit = __ballot(lane < 32 && ((word >> lane) & 1u) && __popc(word & below) == r);
        return 32 * wl + (int)__builtin_ctzll(hit);
    };

    const split::SmallSplit gs = split::small_split(n_exp * (uint32_t)P.gu_tiles, (uint32_t)P.gu_rounds, P.gu_bytes, G);
    const split::SmallSplit sp = DOWN ? split::SmallSplit{n_exp * (uint32_t)P.tiles, 1u} : gs;
    const uint32_t x0 = sp.first(w, G), x1 = sp.first(w + 1, G);
    if (x0 >= x1) return;
    const uint32_t t0 = x0 / sp.per_item, tl = (x1 - 1) / sp.per_item;
    const int n = (int)(tl - t0) + 1;                                     // items of the range
    const int jfirst = sp.per_item == 1 ? 0 : (int)(x0 - t0 * sp.per_item);  // first round of the first item
    const int jlast = sp.per_item == 1 ? J : (int)(x1 - tl * sp.per_item);   // end round of the last item

    // Load cursor: the item whose weights are being issued.
    const int nkb = P.nblocks;
    const int kb0 = nkb * wave / kSWaves, kbe = nkb * (wave + 1) / kSWaves;  // this wavefront's K blocks
    const bool sh_pair = DOWN ? a.down_pair : a.sh_gu_pair, ro_pair = DOWN ? a.down_pair : a.gu_pair;
    int cu = (int)(t0 / (uint32_t)P.tiles), ct = (int)(t0 % (uint32_t)P.tiles), ci = 0;  // expert, tile, item of the range
    rsrc_t ra0, ra1, rs0, rs1;
    uint32_t tstride, toff, kstride;
    auto set_expert = [&](int u) {
        const int e = expert_of(u);
        const bool sh = e < 0, pair = sh ? sh_pair : ro_pair;
        const size_t ee = sh ? 0 : (size_t)e;
        const uint8_t *wa = DOWN ? (sh ? a.sh_down : a.w_down) : (sh ? a.sh_gate : a.w_gate);
        const size_t mat = (size_t)P.mat_bytes * (!DOWN && pair ? 2 : 1);
        ra0 = ra1 = make_rsrc(wa + ee * mat, (uint32_t)mat);
        if (!DOWN && !pair) ra1 = make_rsrc((sh ? a.sh_up : a.w_up) + ee * mat, (uint32_t)mat);
        kstride = pair ? 2 * BLK : BLK;
        tstride = (uint32_t)nkb * BLK * (DOWN || pair ? 2u : 1u);
        toff = pair ? BLK : DOWN ? (uint32_t)nkb * BLK : 0u;
        if constexpr (FMT != FMT_BF16) {
            const uint8_t *s0 = static_cast<const uint8_t *>(DOWN ? (sh ? a.sh_s_down : a.s_down) : (sh ? a.sh_s_gate : a.s_gate));
            const uint8_t *s1 = static_cast<const uint8_t *>(DOWN ? (sh ? a.sh_s_down : a.s_down) : (sh ? a.sh_s_up : a.s_up));
            rs0 = make_rsrc(s0 + ee * P.sc_bytes, P.sc_bytes);
            rs1 = make_rsrc(s1 + ee * P.sc_bytes, P.sc_bytes);
        }
    };
    auto advance = [&]() {
        ++ci;
        if (++ct == P.tiles) {
            ct = 0;
            if (ci < n) set_expert(++cu);
        }
    };

    SmallSlot<FMT> ring[D];
    auto issue = [&](int slot, int j) {
        const int kb = kb0 + j;
        const bool ok = j < J && ci < n && kb < kbe && (ci > 0 || j >= jfirst) && (ci < n - 1 || j < jlast);
        const uint32_t off = (uint32_t)ct * tstride + (uint32_t)kb * kstride + (uint32_t)lane * 16u;
        const uint32_t o0 = ok ? off : kOff, o1 = ok ? off + toff : kOff;
#pragma unroll
        for (int i = 0; i < NV; ++i) ring[slot].v[0][i] = load16<kAuxNT>(ra0, o0 + 1024u * i);
#pragma unroll
        for (int i = 0; i < NV; ++i) ring[slot].v[1][i] = load16<kAuxNT>(ra1, o1 + 1024u * i);
        if constexpr (FMT == FMT_FP8) {  // 128 x 128 block scales: an item's rows lie in one row block
            const uint32_t so = ok ? ((uint32_t)(ct / (DOWN ? 4 : 8)) * (uint32_t)nkb + (uint32_t)kb) * 4u : kOff;
            ring[slot].sc[0] = __builtin_amdgcn_raw_buffer_load_b32(rs0, (int)so, 0, 0);
            ring[slot].sc[1] = DOWN ? ring[slot].sc[0] : __builtin_amdgcn_raw_buffer_load_b32(rs1, (int)so, 0, 0);
        } else if constexpr (FMT == FMT_MXFP4) {
            const uint32_t nq = (uint32_t)((nkb + 3) / 4);
            const uint32_t so = (uint32_t)ct * (DOWN ? 2u : 1u) * nq * 256u + (uint32_t)(kb >> 2) * 256u + (uint32_t)lane * 4u;
            ring[slot].sc[0] = __builtin_amdgcn_raw_buffer_load_b32(rs0, (int)(ok ? so : kOff), 0, 0);
            ring[slot].sc[1] = __builtin_amdgcn_raw_buffer_load_b32(rs1, (int)(ok ? so + (DOWN ? nq * 256u : 0u) : kOff), 0, 0);
        }
    };

    // The current expert's slots and the wavefront's activation blocks (B operands): lane (col, grp) holds
    // token col's elements kb * 128 + 32 grp .. + 31 of each block.
    int myslot = -1, ce = -1;
    bf16x8 bx[J][4];
    const uint32_t brow = (uint32_t)(DOWN ? a.d_ff : a.d) * 2u;
    const rsrc_t rb = make_rsrc(DOWN ? static_cast<const void *>(a.h) : static_cast<const void *>(a.x),
                                (uint32_t)(DOWN ? S + (a.sh_gate ? a.T : 0) : a.T) * brow);
    auto load_b = [&](int u) {
        ce = expert_of(u);
        if (ce < 0) {
            myslot = col < a.T ? S + col : -1;
        } else {
            int cnt = 0;
            for (int base = 0; base < S; base += kWave) {
                const bool hit = base + lane < S && sidx[base + lane] == ce;
                const uint64_t m = __ballot(hit);
                const int r = cnt + __popcll(m & ((1ull << lane) - 1ull));
                if (hit && r < kSmallT) slots[wave][r] = base + lane;
                cnt += __popcll(m);
            }
            __builtin_amdgcn_wave_barrier();  // the same wavefront's LDS accesses stay in order
            myslot = col < cnt ? slots[wave][col] : -1;
        }
        const uint32_t row = (uint32_t)(DOWN ? myslot : ce < 0 ? myslot - S : (int)((uint32_t)myslot / (uint32_t)a.k));
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int k0 = (kb0 + j) * kMacroK + 32 * grp;  // K % 32 == 0: a chunk is all in or all out
            const uint32_t off = myslot >= 0 && kb0 + j < kbe && k0 < P.K ? row * brow + (uint32_t)k0 * 2u : kOff;
#pragma unroll
            for (int s = 0; s < 4; ++s) bx[j][s] = __builtin_bit_cast(bf16x8, load16<0>(rb, off + 16u * s));
        }
        if (DOWN && gs.per_item > 1) {
            // H columns of gate/up items that were cut between workgroups: add their pieces.  A rolled loop:
            // the code is cold and few items are cut (at most one per workgroup boundary).
#pragma unroll 1
            for (int h = 0; h < 2 * J; ++h) {
                const int kb = kb0 + h / 2, n0 = kb * kMacroK + 32 * grp + 16 * (h & 1);  // this lane's 16 columns
                const uint32_t ib = ((uint32_t)u * (uint32_t)P.gu_tiles + (uint32_t)(n0 / 16)) * gs.per_item;
                const bool in = kb < kbe && n0 < P.K;
                const uint32_t w0 = in ? gs.owner(ib, G) : 0u, w1 = in ? gs.owner(ib + gs.per_item - 1, G) : 0u;
                if (w0 == w1) continue;
                f32x4 g[4], up[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const size_t o = (size_t)ce * a.d_ff + n0 + 4 * q;
                    g[q] = ce >= 0 && a.b_gate ? *reinterpret_cast<const f32x4 *>(a.b_gate + o) : f32x4{0.f, 0.f, 0.f, 0.f};
                    up[q] = ce >= 0 && a.b_up ? *reinterpret_cast<const f32x4 *>(a.b_up + o) : f32x4{0.f, 0.f, 0.f, 0.f};
                }
                for (uint32_t v = w0; v <= w1; ++v) {
                    const uint32_t f = gs.first(v, G);
                    if (f >= gs.first(v + 1, G)) continue;  // a workgroup without units
                    const float *src = P.pieces + ((size_t)v * 2 + split::small_piece(f, ib)) * kPieceFloats + col * 4;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        g[q] += *reinterpret_cast<const f32x4 *>(src + 64 * q);
                        up[q] += *reinterpret_cast<const f32x4 *>(src + kPieceFloats / 2 + 64 * q);
                    }
                }
                u32x4 pk[2];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = activate(a, g[q][i], up[q][i]);
                    pk[q >> 1][2 * (q & 1)] = pack_bf16x2(v[0], v[1]);
                    pk[q >> 1][2 * (q & 1) + 1] = pack_bf16x2(v[2], v[3]);
                }
#pragma unroll
                for (int hh = 0; hh < 2 * J; ++hh)
                    if (hh == h && myslot >= 0) {
                        bx[hh / 2][2 * (hh & 1)] = __builtin_bit_cast(bf16x8, pk[0]);
                        bx[hh / 2][2 * (hh & 1) + 1] = __builtin_bit_cast(bf16x8, pk[1]);
                    }
            }
        }
    };

    set_expert(cu);
    int bu = cu, bt = ct;  // expert and tile being contracted
#pragma unroll
    for (int q = 0; q < D - 1; ++q) {
        if (q > 0 && q % JU == 0) advance();
        issue(q, q % JU);
    }
    load_b(bu);

    const bool biased = !DOWN && (a.b_gate != nullptr || a.b_up != nullptr);
    for (int i0 = 0; i0 < n; i0 += PU) {
#pragma unroll
        for (int p = 0; p < PU; ++p) {
            const int i = i0 + p;
            const bool mine = wave == (i & (kSWaves - 1));  // this wavefront finishes the item
            f32x4 gb = f32x4{0.f, 0.f, 0.f, 0.f}, ub = gb;
            if (biased && mine && i < n && ce >= 0) {
                const size_t o = (size_t)ce * a.d_ff + 16 * bt + 4 * grp;
                if (a.b_gate) gb = *reinterpret_cast<const f32x4 *>(a.b_gate + o);
                if (a.b_up) ub = *reinterpret_cast<const f32x4 *>(a.b_up + o);
            }
            f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
            const int jl = i == 0 ? jfirst : 0, jh = i == n - 1 ? jlast : J;
#pragma unroll
            for (int j = 0; j < JU; ++j) {
                const int q = p * JU + j + D - 1;  // the round whose loads go out now
                if (q % JU == 0) advance();
                issue(q % D, q % JU);
                if (j < J && i < n && j >= jl && j < jh) {
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
            if (i < n) {
                const int buf = i & 1;
                red[buf][wave][0][lane] = acc[0];
                red[buf][wave][1][lane] = acc[1];
                // LDS only: the weight loads in flight stay in flight.  An item's sums are read before the
                // next item's barrier and overwritten after it.
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                if (mine) {
                    f32x4 r0 = red[buf][0][0][lane], r1 = red[buf][0][1][lane];
#pragma unroll
                    for (int v = 1; v < kSWaves; ++v) {
                        r0 += red[buf][v][0][lane];
                        r1 += red[buf][v][1][lane];
                    }
                    if (DOWN) {
                        if (myslot >= 0) {
                            float *dst = a.o + (size_t)myslot * a.d + 32 * bt + 4 * grp;
                            *reinterpret_cast<f32x4 *>(dst) = r0;
                            *reinterpret_cast<f32x4 *>(dst + 16) = r1;
                        }
                    } else if (jl == 0 && jh == J) {
                        if (myslot >= 0) {
                            r0 += gb;
                            r1 += ub;
                            float h[4];
#pragma unroll
                            for (int r = 0; r < 4; ++r) h[r] = activate(a, r0[r], r1[r]);
                            *reinterpret_cast<u32x2 *>(a.h + (size_t)myslot * a.d_ff + 16 * bt + 4 * grp) =
                                u32x2{pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3])};
                        }
                    } else {
                        float *dst = P.pieces + ((size_t)w * 2 + (jl > 0 ? 0 : 1)) * kPieceFloats + lane * 4;
                        *reinterpret_cast<f32x4 *>(dst) = r0;
                        *reinterpret_cast<f32x4 *>(dst + kPieceFloats / 2) = r1;
                    }
                }
                if (++bt == P.tiles) {
                    bt = 0;
                    if (i + 1 < n) load_b(++bu);
                }
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

template <int FMT, bool DOWN>
static hipError_t launch_projection(const SmallParams &p, hipStream_t stream)
{
    const dim3 grid(p.workers), block(kSThreads);
    switch ((p.nblocks + kSWaves - 1) / kSWaves) {
#define SMALL_CASE(J)                                                                          \
    case J:                                                                                    \
        hipLaunchKernelGGL((expert_small_kernel<FMT, DOWN, J>), grid, block, 0, stream, p);    \
        break;
        SMALL_CASE(1) SMALL_CASE(2) SMALL_CASE(3) SMALL_CASE(4) SMALL_CASE(5) SMALL_CASE(6) SMALL_CASE(7) SMALL_CASE(8)
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
    const uint64_t n_exp = (uint64_t)(a.E < a.T * a.k ? a.E : a.T * a.k) + 1;
    const uint64_t units = n_exp * ((uint64_t)(a.d_ff / 16) * ((nu + kSWaves - 1) / kSWaves) + a.d / 32);
    return units * (uint64_t)workers < (1ull << 31);
}

template <int FMT>
static hipError_t launch_small_fmt(const VerifyArgs &args, uint8_t *ws_base, const VerifyWorkspace &ws, hipStream_t stream,
                                   hipEvent_t const *events)
{
    auto mark = [&](int i) { return events && events[i] ? hipEventRecord(events[i], stream) : hipSuccess; };
    SmallParams p{};
    p.a = args;
    p.a.h = reinterpret_cast<uint16_t *>(ws_base + ws.h_offset);
    p.a.o = reinterpret_cast<float *>(ws_base + ws.o_offset);
    p.workers = ws.workers;
    p.pieces = reinterpret_cast<float *>(ws_base + ws.p_offset);
    const VerifyArgs &a = p.a;
    p.N = a.d_ff;
    p.K = a.d;
    p.nblocks = (a.d + kMacroK - 1) / kMacroK;
    p.tiles = a.d_ff / 16;
    p.mat_bytes = (uint32_t)packed_matrix_bytes(FMT, a.d_ff, a.d);
    p.sc_bytes = (uint32_t)packed_scale_bytes(FMT, a.d_ff, a.d);
    p.gu_tiles = p.tiles;
    p.gu_rounds = (p.nblocks + kSWaves - 1) / kSWaves;
    p.gu_bytes = (uint32_t)p.nblocks * 2048u * Fmt<FMT>::kVecs;
    hipError_t err;
    if ((err = mark(0)) != hipSuccess) return err;
    if ((err = launch_projection<FMT, false>(p, stream)) != hipSuccess) return err;
    if ((err = mark(1)) != hipSuccess) return err;
    p.N = a.d;
    p.K = a.d_ff;
    p.nblocks = (a.d_ff + kMacroK - 1) / kMacroK;
    p.tiles = a.d / 32;
    p.mat_bytes = (uint32_t)packed_matrix_bytes(FMT, a.d, a.d_ff);
    p.sc_bytes = (uint32_t)packed_scale_bytes(FMT, a.d, a.d_ff);
    if ((err = mark(2)) != hipSuccess) return err;
    if ((err = launch_projection<FMT, true>(p, stream)) != hipSuccess) return err;
    if ((err = mark(3)) != hipSuccess) return err;
    hipLaunchKernelGGL(combine_small_kernel, dim3((a.T * (a.d / 4) + 255) / 256 + 1), dim3(256), 0, stream, p.a);
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
