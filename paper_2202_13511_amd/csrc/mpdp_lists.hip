// The levels of the block-based path as lists of connected sets (see
// mpdp_lists.h): one launch per level evaluates the level's sets and grows
// the next level's list.
#include <hip/hip_runtime.h>

#include "mpdp_internal.h"
#include "mpdp_lists.h"

namespace mpdp {
namespace {

// Levels with at least this many members per set share a set among several
// waves when they have fewer sets than waves: below, a set has too few pairs
// to divide.
constexpr uint32_t kShareMinK = 10;

// One workgroup of 16 waves per CU (the waves' pools, the rank table and the
// query fill 160 KB of LDS).  The next level's list first, which the
// workgroup does in step, then each wave its own sets.  `tally` holds two
// sums per workgroup (pairs, Alg. 3 candidates): adding them to one counter
// per wave took longer than most levels.
template <int CM>
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
    // sets per wave at a time: the same for all waves, so that none goes
    // another round for the last few sets
    const uint32_t rounds = (count + 64u * nw - 1u) / (64u * nw);
    const uint32_t per = (count + rounds * nw - 1u) / (rounds * nw);
    uint32_t group = 1u;  // lanes that grow one set's successors
    while (group < 16u && count * group < 32u * nw) group <<= 1;
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
        expand_sets(L, list, count, next, &cnt->level_count[k + 1], w, nw, group, reinterpret_cast<uint32_t *>(buf),
                    sizeof(buf) / 4, ends, lane);
    unsigned long long ccp = 0, evaluated = 0;
    eval_pairs<CM>(L, ranks, n > 24u, M, list, count, k, w, nw, per, parts, buf[threadIdx.x >> 6],
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
    if (threadIdx.x < 2) tally[2 * blockIdx.x + threadIdx.x] += sums[threadIdx.x];
}

}  // namespace

hipError_t launch_level_pairs(const DevGraph *g, int cost_model, uint32_t n, uint32_t k, const uint32_t *list,
                              uint32_t *next, Counters *cnt, MemoPtrs memo, HeavyPart *rec, uint32_t *arrived,
                              unsigned long long *tally, hipStream_t s) {
    if (cost_model == MPDP_COST_COUT)
        hipLaunchKernelGGL(k_level_pairs<MPDP_COST_COUT>, dim3(kPairGrid), dim3(kPairBlock), 0, s, g, n, k, list, next,
                           cnt, memo, rec, arrived, tally);
    else
        hipLaunchKernelGGL(k_level_pairs<MPDP_COST_PGLIKE>, dim3(kPairGrid), dim3(kPairBlock), 0, s, g, n, k, list,
                           next, cnt, memo, rec, arrived, tally);
    return hipGetLastError();
}

}  // namespace mpdp
