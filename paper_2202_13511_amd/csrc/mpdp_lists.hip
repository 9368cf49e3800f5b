// Levels as lists of connected sets (see mpdp_lists.h), of cyclic queries from
// 19 relations on and of tree joins: one launch per level evaluates the level's
// sets and grows the next level's list.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mpdp_internal.h"
#include "mpdp_lists.h"

namespace mpdp {
namespace {

// Levels with at least this many members per set share a set among several
// waves when they have fewer sets than waves: below, a set has too few pairs
// to divide.
constexpr uint32_t kShareMinK = 10;

// PG-like levels whose pairs' cards are read only where the costs leave a
// chance (see pass_pair): those bound by their gathers, of many sets or of which
// most subsets are connected and make pairs.  Other levels wait for each step of
// the search, and a pair takes one more with its cards read later (2 to 6 %).
// Asked only (lazy_query) where a memo's costs are more than the L2s hold (8 B <<
// n: 32 MB at 22 relations) or the graph has many edges: a smaller star's sets
// have one pair a member.  Always later / always along with the costs / by this
// rule, ms: cliques of 19 4.7 / 8.2 / 5.0, of 22 245 / 604 / 257; two hubs of 20
// relations 69 / 160 / 74; cycles with chords, of 24 (8) 1.77 / 1.68 / 1.69, 24 (14)
// 3.47 / 4.14 / 3.43, 28 (10) 5.08 / 6.13 / 5.06, 30 (11) 10.9 / 15.4 / 10.9; star
// of 22 with two more edges 1.20 / 1.12 / 1.12, of 24 with three 4.07 / 4.40 / 4.07;
// chain of 16 on a clique of 14 3.66 / 3.35 / 3.42.
__device__ __forceinline__ bool lazy_level(uint32_t count, uint64_t subsets) {
    return count >= 65536u || (count >= 2048u && 4ull * count >= subsets);
}

// One workgroup of 16 waves per CU (the waves' pools, the rank table and the
// query fill 160 KB of LDS).  The next level's list first, which the
// workgroup does in step, then each wave its own sets.  `tally` holds two
// sums per workgroup (pairs, Alg. 3 candidates): adding them to one counter
// per wave took longer than most levels.
template <int CM, bool kWide, bool kLazy>
__global__ __launch_bounds__(kPairBlock) void k_level_pairs(const DevGraph *g, uint32_t n, uint32_t k,
                                                            const uint32_t *list, uint32_t *next, Counters *cnt,
                                                            MemoPtrs M, HeavyPart *rec, uint32_t *arrived,
                                                            unsigned long long *tally) {
    __shared__ __align__(16) unsigned char image[kListLdsBytes];
    __shared__ __align__(16) uint32_t ranks[kRankWords];
    __shared__ __align__(16) PairBuf buf[kPairBlock / 64];
    __shared__ ExpandEnds ends;
    __shared__ unsigned long long sums[2];
    const uint32_t count = cnt->level_count[k];
    const uint32_t nw = gridDim.x * (kPairBlock / 64);
    const uint32_t per = pair_sets(count, nw);
    const uint32_t group = expand_group(count, 64u * nw);
    const uint32_t parts = k >= kShareMinK && 2u * count <= nw ? min(64u, nw / count) : 1u;
    // neighbouring items to different CUs, so that few items still fill the chip
    const uint32_t lane = threadIdx.x & 63u, w = (threadIdx.x >> 6) * gridDim.x + blockIdx.x;
    const uint32_t items = parts > 1u ? count * parts : (count + per - 1u) / per;
    if (blockIdx.x >= items && blockIdx.x * (64u / group) >= count) return;  // the whole workgroup
    LdsGraph &L = *reinterpret_cast<LdsGraph *>(image);
    stage_graph_prefix(g, L, kListLdsBytes);
    stage_ranks(ranks, n);
    if (threadIdx.x < 2) sums[threadIdx.x] = 0ull;
    __syncthreads();
    if (k < n)
        expand_sets<kWide>(L, list, count, next, &cnt->level_count[k + 1], w, nw, group, reinterpret_cast<uint32_t *>(buf),
                    sizeof(buf) / 4, ends, lane);
    unsigned long long ccp = 0, evaluated = 0;
    const ColexMemo at{ranks, L.loff, kWide};
    const PairParts pp{rec, arrived};
    if (kLazy && lazy_level(count, L.loff[k + 1] - L.loff[k]))
        eval_pairs<CM, kWide, true>(L, at, M, list, count, k, w, nw, per, parts, buf[threadIdx.x >> 6], pp, lane, ccp, evaluated);
    else
        eval_pairs<CM, kWide, false>(L, at, M, list, count, k, w, nw, per, parts, buf[threadIdx.x >> 6], pp, lane, ccp, evaluated);
    for (int off = 32; off >= 1; off >>= 1) {
        ccp += (unsigned long long)__shfl_xor((long long)ccp, off);
        evaluated += (unsigned long long)__shfl_xor((long long)evaluated, off);
    }
    if (lane == 0) {
        atomicAdd(&sums[0], ccp);
        atomicAdd(&sums[1], evaluated);
    }
    __syncthreads();
    if (threadIdx.x < 2) tally[2 * blockIdx.x + threadIdx.x] += sums[threadIdx.x];
}

// Dense queries of up to 24 relations: no plan yet for any set.
__global__ __launch_bounds__(256) void k_no_plans(double *cost, uint64_t sets) {
    double2 *c = reinterpret_cast<double2 *>(cost);
    for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < sets / 2; i += gridDim.x * 256ull) c[i] = make_double2(-1.0, -1.0);
}

// One level of them: the next level's list, then every set's subsets.  Two
// workgroups of 16 waves per CU (their rank tables and queries fill its LDS).
// Bound by the gathers past the L2 and the eight table lookups of a candidate's
// two ranks: a clique of 22 takes 113 ms, 138 G pairs a second (searched 239, and
// 222 when each block's subsets were walked).
constexpr int kWalkBlock = 1024;
constexpr uint32_t kWalkGrid = 512;
template <int CM>
__global__ __launch_bounds__(kWalkBlock) void k_level_walk(const DevGraph *g, uint32_t n, uint32_t k,
                                                           const uint32_t *list, uint32_t *next, Counters *cnt,
                                                           MemoPtrs M, HeavyPart *rec, uint32_t *arrived,
                                                           unsigned long long *tally) {
    __shared__ __align__(16) unsigned char image[kListLdsBytes];
    __shared__ __align__(16) uint32_t ranks[kRankWords24];
    __shared__ __align__(16) uint32_t todo[kWalkBlock / 64][64 * 12];  // (block_candidates: 24 relations, 12 pieces)
    __shared__ ExpandEnds ends;
    __shared__ unsigned long long sums[2];
    const uint32_t count = cnt->level_count[k];
    const uint32_t nw = gridDim.x * (kWalkBlock / 64);
    const uint32_t per = pair_sets(count, nw), group = expand_group(count, 64u * nw);
    const uint32_t most = min(nw, kPairWaves), parts = k >= kShareMinK && 2u * count <= most ? min(64u, most / count) : 1u;
    const uint32_t lane = threadIdx.x & 63u, w = (threadIdx.x >> 6) * gridDim.x + blockIdx.x;
    const uint32_t items = parts > 1u ? count * parts : (count + per - 1u) / per;
    if (blockIdx.x >= items && blockIdx.x * (64u / group) >= count) return;  // the whole workgroup
    LdsGraph &L = *reinterpret_cast<LdsGraph *>(image);
    stage_graph_prefix(g, L, kListLdsBytes);
    stage_ranks(ranks, 24u);
    if (threadIdx.x < 2) sums[threadIdx.x] = 0ull;
    __syncthreads();
    if (k < n)
        expand_sets<false>(L, list, count, next, &cnt->level_count[k + 1], w, nw, group, &todo[0][0], sizeof(todo) / 4, ends, lane);
    unsigned long long ccp = 0, evaluated = 0;
    eval_subsets<CM>(L, ColexMemo{ranks, L.loff, false}, M, list, count, k, w, nw, per, parts, todo[threadIdx.x >> 6],
                     PairParts{rec, arrived}, lane, ccp, evaluated);
    for (int off = 32; off >= 1; off >>= 1) {
        ccp += (unsigned long long)__shfl_xor((long long)ccp, off);
        evaluated += (unsigned long long)__shfl_xor((long long)evaluated, off);
    }
    if (lane == 0) {
        atomicAdd(&sums[0], ccp);
        atomicAdd(&sums[1], evaluated);
    }
    __syncthreads();
    if (threadIdx.x < 2) atomicAdd(&tally[2u * (blockIdx.x % kPairGrid) + threadIdx.x], sums[threadIdx.x]);
}

// One level of a tree join: the first `eval` workgroups cost the level's
// sets, the others grow the next level's list, so that neither waits for the
// other's reads.
constexpr int kTreeBlock = 256;
constexpr uint32_t kTreeExpand = 4096;  // words of the expansion's LDS buffer

template <int CM>
__global__ __launch_bounds__(kTreeBlock) void k_tree_level(const DevGraph *g, uint32_t n, uint32_t k, uint32_t eval,
                                                           const uint32_t *list, uint32_t *next, Counters *cnt,
                                                           MemoPtrs M) {
    __shared__ __align__(16) LdsGraph L;
    __shared__ __align__(16) uint32_t ranks[kRankWords > kTreeExpand ? kRankWords : kTreeExpand];
    __shared__ ExpandEnds ends;
    const uint32_t count = cnt->level_count[k], lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    stage_graph_preorder(g, L);
    if (blockIdx.x < eval) {
        stage_ranks(ranks, n);
        __syncthreads();
        const uint32_t threads = eval * kTreeBlock;
        eval_tree_list<CM>(L, ColexMemo{ranks, L.loff, n > 24u}, M, list, count, k, tree_group(count, threads),
                           (wave * eval + blockIdx.x) * 64u + lane, threads);
    } else {
        const uint32_t blocks = gridDim.x - eval, threads = blocks * kTreeBlock;
        expand_tree(L, list, count, next, &cnt->level_count[k + 1], wave * blocks + blockIdx.x - eval, threads / 64,
                    ranks, kTreeExpand, ends, lane);
    }
}

// Levels k0 .. k1 of a tree join by one workgroup, barriers between them:
// levels of a few thousand pairs take less time than a launch.  The span that
// starts at level 2 also fills the base relations and level 2's list (and
// needs no k_init).  kStar: a star around relation 0, of which every set that
// holds it is connected; each level's list is unranked, so that the span
// needs none from the level before.
constexpr int kSpanBlock = 1024;
constexpr uint32_t kSpanExpand = 16384;

template <int CM, bool kStar>
__global__ __launch_bounds__(kSpanBlock) void k_tree_span(const DevGraph *src, DevGraph *g, uint32_t n, uint32_t k0,
                                                          uint32_t k1, uint32_t *even, uint32_t *odd, Counters *cnt,
                                                          MemoPtrs M) {
    __shared__ __align__(16) DevGraph G;
    __shared__ __align__(16) uint32_t ranks[kRankWords];
    __shared__ uint32_t buf[kSpanExpand];
    __shared__ ExpandEnds ends;
    __shared__ uint32_t counts[36];  // sets of level k, while the span lasts
    const uint32_t t = threadIdx.x;
    const LdsGraph &L = G.lds;
    if (t < 36u) counts[t] = t != k0 || kStar ? 0u : k0 == 2u ? n - 1u : cnt->level_count[k0];
    bring_graph(k0 == 2u ? src : nullptr, g, G);
    stage_ranks(ranks, n);
    if (k0 == 2u) {
        uint32_t *words = reinterpret_cast<uint32_t *>(cnt);
        for (uint32_t i = t; i < sizeof(Counters) / 4; i += blockDim.x)
            words[i] = i == offsetof(Counters, level_count) / 4 + 2 ? n - 1u : 0u;
    }
    __syncthreads();
    if (k0 == 2u && t < n) {
        const uint64_t at = L.loff[1] + t;
        M.cost[at] = L.bcost[t];
        M.card[at] = L.card[t];
        M.left[at] = 0;
        M.op[at] = MPDP_OP_SCAN;
    }
    if (!kStar && k0 == 2u && t >= 64u && t - 64u < n) first_tree_list(L, t - 64u, even);
    __syncthreads();
    for (uint32_t k = k0; k <= k1; ++k) {
        uint32_t *list = (k & 1u) ? odd : even;
        const uint32_t count = kStar ? L.binom[(n - 1u) * 33u + k - 1u] : counts[k];
        if (kStar) {
            if (t == 0) cnt->level_count[k] = count;
            for (uint32_t i = t; i < count; i += kSpanBlock)
                list[i] = (colex_unrank(L.binom, (int)n - 1, (int)k - 1, i) << 1) | 1u;
            __syncthreads();
        } else if (k < n) {
            expand_tree(L, list, count, (k & 1u) ? even : odd, &counts[k + 1], t >> 6, kSpanBlock / 64, buf, kSpanExpand,
                        ends, t & 63u);
            if (t == 0) cnt->level_count[k + 1] = counts[k + 1];
        }
        eval_tree_list<CM>(L, ColexMemo{ranks, L.loff, n > 24u}, M, list, count, k, tree_group(count, kSpanBlock), t, kSpanBlock);
        __syncthreads();
    }
}

}  // namespace

// Which queries take the kernel that holds both forms of the search: it costs
// 1 to 1.7 % where no level gains (cycle of 28 912 us / 923, of 28 with two chords
// 1138 / 1158), as where up to three edges more than a tree's meet no relation of
// five or more (star of 24 with one more edge 4152 / 3907).
bool lazy_query(uint32_t n, uint32_t m, const uint32_t *adj) {
    if (many_edges(n, m)) return true;
    if (n < 23) return false;
    const auto hub = [](uint32_t a) { return __builtin_popcount(a) > 4; };
    return m >= n + 3 || std::any_of(adj, adj + n, hub);
}

hipError_t launch_level_pairs(const DevGraph *g, int cost_model, bool lazy, uint32_t n, uint32_t k,
                              const uint32_t *list, uint32_t *next, Counters *cnt, MemoPtrs memo, HeavyPart *rec,
                              uint32_t *arrived, unsigned long long *tally, hipStream_t s) {
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(kPairGrid), dim3(kPairBlock), 0, s, g, n, k, list, next, cnt, memo, rec,
                           arrived, tally);
    };
    if (cost_model == MPDP_COST_COUT)
        n > 24 ? go(k_level_pairs<MPDP_COST_COUT, true, false>) : go(k_level_pairs<MPDP_COST_COUT, false, false>);
    else if (lazy)
        n > 24 ? go(k_level_pairs<MPDP_COST_PGLIKE, true, true>) : go(k_level_pairs<MPDP_COST_PGLIKE, false, true>);
    else
        n > 24 ? go(k_level_pairs<MPDP_COST_PGLIKE, true, false>) : go(k_level_pairs<MPDP_COST_PGLIKE, false, false>);
    return hipGetLastError();
}

hipError_t launch_no_plans(MemoPtrs memo, uint32_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_no_plans, dim3(1024), dim3(256), 0, s, memo.cost, 1ull << n);
    return hipGetLastError();
}

hipError_t launch_level_walk(const DevGraph *g, int cost_model, uint32_t n, uint32_t k, const uint32_t *list,
                             uint32_t *next, Counters *cnt, MemoPtrs memo, HeavyPart *rec, uint32_t *arrived,
                             unsigned long long *tally, hipStream_t s) {
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(kWalkGrid), dim3(kWalkBlock), 0, s, g, n, k, list, next, cnt, memo, rec, arrived,
                           tally);
    };
    cost_model == MPDP_COST_COUT ? go(k_level_walk<MPDP_COST_COUT>) : go(k_level_walk<MPDP_COST_PGLIKE>);
    return hipGetLastError();
}

hipError_t launch_tree_level(const DevGraph *g, int cost_model, uint32_t n, uint32_t k, uint64_t count,
                             const uint32_t *list, uint32_t *next, Counters *cnt, MemoPtrs memo, hipStream_t s) {
    // eight lanes a set, up to four workgroups per CU; one lane a set to grow
    // the list, up to one workgroup per CU
    const uint32_t eval = (uint32_t)std::min<uint64_t>((count * 8 + kTreeBlock - 1) / kTreeBlock, kTreeListGrid);
    const uint32_t grid = eval + (k < n ? (uint32_t)std::min<uint64_t>((count + kTreeBlock - 1) / kTreeBlock, 256) : 0u);
    if (cost_model == MPDP_COST_COUT)
        hipLaunchKernelGGL(k_tree_level<MPDP_COST_COUT>, dim3(grid), dim3(kTreeBlock), 0, s, g, n, k, eval, list, next,
                           cnt, memo);
    else
        hipLaunchKernelGGL(k_tree_level<MPDP_COST_PGLIKE>, dim3(grid), dim3(kTreeBlock), 0, s, g, n, k, eval, list,
                           next, cnt, memo);
    return hipGetLastError();
}

hipError_t launch_tree_span(const DevGraph *src, DevGraph *g, int cost_model, bool star, uint32_t n, uint32_t k0,
                            uint32_t k1, uint32_t *even, uint32_t *odd, Counters *cnt, MemoPtrs memo, hipStream_t s) {
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kSpanBlock), 0, s, src, g, n, k0, k1, even, odd, cnt, memo);
    };
    if (cost_model == MPDP_COST_COUT)
        star ? go(k_tree_span<MPDP_COST_COUT, true>) : go(k_tree_span<MPDP_COST_COUT, false>);
    else
        star ? go(k_tree_span<MPDP_COST_PGLIKE, true>) : go(k_tree_span<MPDP_COST_PGLIKE, false>);
    return hipGetLastError();
}

}  // namespace mpdp
