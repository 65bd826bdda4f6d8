// Expert union, histogram, scans and stable grouping on gfx950, by one
// workgroup of 1024 threads (E <= 1024, so thread e owns expert e).
//
// The routed slots are taken 1024 at a time, one per thread, in slot order
// (wavefront w holds slots 64w .. 64w + 63 of a pass).  Within a wavefront,
// lanes holding the same expert find each other with one ballot per bit of
// the expert id; a lane's rank among the lower such lanes orders equal
// experts by slot, and the highest lane of each expert records the
// wavefront's count in LDS.  Per expert, the counts of the earlier passes and
// wavefronts plus the rank place every slot.  So the grouping is a stable
// counting sort by expert.
//
// Up to 4096 slots (a verification batch of 512 tokens x 8) every pass stays in
// registers: the slots are loaded and matched once, the counts of all passes
// lie side by side in LDS, and one pass of scans gives first grouped and union
// positions (one scan of both: slots and used experts below 2^16).  At 1600
// slots, union and token-group plan in one launch: 5.9 us; the union alone took
// 8.4 us with the separate counting and placement sweeps that larger batches
// keep, which load and match every slot twice.  A single pass (1024 slots) keeps
// its counts in 32 bits: 16-bit LDS accesses and a scan each for slots and
// experts took 0.3 us more (E = 256, 512 slots: 3.6 us, now 3.3).
#pragma once

#include <type_traits>

#include "device.hpp"

namespace ecospec {

constexpr int kUnionThreads = 1024;
constexpr int kUnionWaves = kUnionThreads / kWave;
constexpr int kUnionPasses = 4;  // passes held in registers

struct UnionLds {
    union {
        uint16_t wcnt16[kUnionPasses][kUnionWaves][kUnionThreads];  // per-pass, per-wavefront counts, then positions
        int wcnt[kUnionWaves][kUnionThreads];                       // of the only, or (beyond kUnionPasses) the current pass
    };
    int member_id[kUnionThreads];
    int member_start[kUnionThreads];
    int wave_tot[2 * kUnionWaves];
    int U, placed;  // distinct experts, placed slots
};

// What the scans found, into the routing arrays and LDS: thread e holds expert e's count, union position and
// first grouped position.
__device__ __forceinline__ void union_members(UnionLds &L, int E, int c, int pos, int start, int U, int placed,
                                              int32_t *__restrict__ counts)
{
    const int tid = threadIdx.x;
    if (tid < E) {
        counts[tid] = c;
        if (c > 0) {
            L.member_id[pos] = tid;
            L.member_start[pos] = start;
        }
    }
    if (tid == 0) {
        L.U = U;
        L.placed = placed;
    }
}

__device__ __forceinline__ void union_write(const UnionLds &L, int E, int U, int placed, int32_t *__restrict__ union_ids,
                                            int32_t *__restrict__ n_unique, int32_t *__restrict__ offsets)
{
    for (int u = threadIdx.x; u <= E; u += kUnionThreads) {
        if (u < E) union_ids[u] = u < U ? L.member_id[u] : -1;
        offsets[u] = u < U ? L.member_start[u] : placed;
    }
    if (threadIdx.x == 0) *n_unique = U;
}

// S <= PASSES * 1024 slots.
template <int PASSES>
__device__ __forceinline__ void union_in_registers(UnionLds &L, const int32_t *__restrict__ idx, int S, int E, int nbits,
                                                   int32_t *__restrict__ counts, int32_t *__restrict__ union_ids,
                                                   int32_t *__restrict__ n_unique, int32_t *__restrict__ offsets,
                                                   int32_t *__restrict__ perm)
{
    using count_t = std::conditional_t<PASSES == 1, int, uint16_t>;
    auto at = [&](int p, int w, int e) -> count_t & {
        if constexpr (PASSES == 1) return L.wcnt[w][e];
        else return L.wcnt16[p][w][e];
    };
    const int tid = threadIdx.x, wave = tid / kWave;
    int e[PASSES], rank[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) e[p] = p * kUnionThreads + tid < S ? idx[p * kUnionThreads + tid] : -1;
    if (tid < E)
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            for (int w = 0; w < kUnionWaves; ++w) at(p, w, tid) = 0;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        bool top;
        int cnt;
        wave_match(e[p], (unsigned)e[p] < (unsigned)E, nbits, rank[p], top, cnt);
        if (top) at(p, wave, e[p]) = (count_t)cnt;
    }
    __syncthreads();
    int c = 0;
    if (tid < E)
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            for (int w = 0; w < kUnionWaves; ++w) c += at(p, w, tid);
    static_assert(kUnionPasses * kUnionThreads < 1 << 15, "slots and experts in one word");
    int tot = 0;
    const int ex = block_exclusive_scan((c << 16) | (c > 0 ? 1 : 0), L.wave_tot, &tot);
    const int pos = ex & 0xffff, start = ex >> 16, U = tot & 0xffff, placed = tot >> 16;
    union_members(L, E, c, pos, start, U, placed, counts);
    if (tid < E) {  // counts -> first position of each pass's and wavefront's slots (below 4096)
        int run = start;
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            for (int w = 0; w < kUnionWaves; ++w) {
                const int n = at(p, w, tid);
                at(p, w, tid) = (count_t)run;
                run += n;
            }
    }
    __syncthreads();
    union_write(L, E, U, placed, union_ids, n_unique, offsets);
#pragma unroll
    for (int p = 0; p < PASSES; ++p)
        if ((unsigned)e[p] < (unsigned)E) perm[at(p, wave, e[p]) + rank[p]] = p * kUnionThreads + tid;
}

// The union, scans and grouping of S routed slots idx[0 .. S), by the whole 1024-thread workgroup; U, placed and
// the members' first positions stay in L (behind no barrier).
__device__ __forceinline__ void union_block(UnionLds &L, const int32_t *__restrict__ idx, int S, int E,
                                            int32_t *__restrict__ counts, int32_t *__restrict__ union_ids,
                                            int32_t *__restrict__ n_unique, int32_t *__restrict__ offsets,
                                            int32_t *__restrict__ perm)
{
    const int tid = threadIdx.x, wave = tid / kWave;
    int nbits = 0;
    while ((1 << nbits) < E) ++nbits;
    const int passes = (S + kUnionThreads - 1) / kUnionThreads;
    if (passes == 1)
        return union_in_registers<1>(L, idx, S, E, nbits, counts, union_ids, n_unique, offsets, perm);
    if (passes == 2)
        return union_in_registers<2>(L, idx, S, E, nbits, counts, union_ids, n_unique, offsets, perm);
    if (passes <= kUnionPasses)
        return union_in_registers<kUnionPasses>(L, idx, S, E, nbits, counts, union_ids, n_unique, offsets, perm);

    // 1. Counts: per-wavefront matches, summed per expert over wavefronts and passes.
    int total = 0;  // thread e: slots routed to expert e
    for (int ps = 0; ps < passes; ++ps) {
        for (int w = 0; w < kUnionWaves; ++w) L.wcnt[w][tid] = 0;
        __syncthreads();
        const int s = ps * kUnionThreads + tid;
        const int e = s < S ? idx[s] : -1;
        const bool ok = (unsigned)e < (unsigned)E;
        int rank, cnt;
        bool top;
        wave_match(e, ok, nbits, rank, top, cnt);
        if (top) L.wcnt[wave][e] = cnt;
        __syncthreads();
        if (tid < E)
            for (int w = 0; w < kUnionWaves; ++w) total += L.wcnt[w][tid];
        __syncthreads();
    }

    // 2. Union positions and first grouped positions.
    const int c = tid < E ? total : 0;
    int pos, start, U, placed;
    block_exclusive_scan2(c > 0 ? 1 : 0, c, L.wave_tot, pos, start, U, placed);
    union_members(L, E, c, pos, start, U, placed, counts);
    __syncthreads();
    union_write(L, E, U, placed, union_ids, n_unique, offsets);

    // 3. Placement, pass by pass: thread e turns the per-wavefront counts into
    //    first positions (in place), then every slot of the pass is placed.
    int run = start;  // thread e: next position of expert e
    for (int ps = 0; ps < passes; ++ps) {
        for (int w = 0; w < kUnionWaves; ++w) L.wcnt[w][tid] = 0;
        __syncthreads();
        const int s = ps * kUnionThreads + tid;
        const int e = s < S ? idx[s] : -1;
        const bool ok = (unsigned)e < (unsigned)E;
        int rank, cnt;
        bool top;
        wave_match(e, ok, nbits, rank, top, cnt);
        if (top) L.wcnt[wave][e] = cnt;
        __syncthreads();
        if (tid < E) {
            for (int w = 0; w < kUnionWaves; ++w) {
                const int n = L.wcnt[w][tid];
                L.wcnt[w][tid] = run;
                run += n;
            }
        }
        __syncthreads();
        if (ok) perm[L.wcnt[wave][e] + rank] = s;
        __syncthreads();
    }
}

}  // namespace ecospec
