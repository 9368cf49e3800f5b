// Cyclic queries of up to kBitsMaxRel relations: the connectivity of every
// relation set is computed once, as a bitmap that fits a workgroup's LDS, and
// a level tests all subsets of its sets against it.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mpdp_internal.h"
#include "mpdp_lists.h"

namespace mpdp {
namespace {

constexpr int kBitsInitBlock = 1024, kBitsBlock = 256;
constexpr uint32_t kBitsGrid = 2048;

// One thread per relation set: connectivity into the bitmap, connected sets
// into their level's list (from loff[k]), their cards, and the entries of
// single relations.
__global__ __launch_bounds__(kBitsInitBlock) void k_bits_init(const DevGraph *g, uint32_t n, Counters *cnt,
                                                              BitsSpace B) {
    __shared__ __align__(16) unsigned char image[kListLdsBytes];
    __shared__ uint32_t have[kBitsMaxRel + 1], start[kBitsMaxRel + 1];
    LdsGraph &L = *reinterpret_cast<LdsGraph *>(image);
    const uint32_t t = threadIdx.x, S = blockIdx.x * kBitsInitBlock + t;
    stage_graph_prefix(g, L, kListLdsBytes);
    if (t <= n) have[t] = 0;
    __syncthreads();
    const bool in = S != 0u && (S >> n) == 0u;
    const uint32_t k = (uint32_t)popc32(S);
    bool conn = false;
    if (in) {
        uint32_t seen = lowbit(S), fr = seen;
        while (fr != 0u) {
            fr = nbrs_of<false>(L.nb, fr) & S & ~seen;
            seen |= fr;
        }
        conn = seen == S;
    }
    const unsigned long long m = __ballot(conn);
    if ((t & 31u) == 0u && (S >> n) == 0u) B.conn[S >> 5] = (uint32_t)(m >> (t & 32u));
    uint32_t at = 0;
    if (conn && k >= 2u) at = atomicAdd(&have[k], 1u);
    __syncthreads();
    if (t >= 2u && t <= n && have[t]) start[t] = atomicAdd(&cnt->level_count[t], have[t]);
    if (conn) {
        B.card[(size_t)S * B.stride] = k == 1u ? L.card[ctz32(S)] : card_of(L, S);
        if (k == 1u) {
            B.cost[(size_t)S * B.stride] = L.bcost[ctz32(S)];
            B.cand[S] = 0;
        }
    }
    __syncthreads();
    if (conn && k >= 2u) B.list[L.loff[k] + start[k] + at] = S;
}

// One level.  A set's candidates are its subsets that hold its lowest
// relation, A = lowest + x, and the pair (A, S - A) counts if the bitmap has
// both: two LDS reads a candidate, none waiting for another, where the search
// of larger queries (eval_pairs) takes a chain of some 3 000 cycles a pair.
// All 3^n / 2 candidates of 17 relations take some 60 us of the whole chip,
// less than 17 levels of such chains.  2^lgP lanes take a set of up to six
// relations, a candidate each; from seven on a wave takes a set, or, on levels
// of few sets, several waves one, whose best keys meet in `rec` (as in
// eval_pairs).  Where few candidates count, they are collected until there is
// one for every lane.  Costs are read from an array indexed by the set (8 B
// << n, in the L2), under PG-like with the cards as one 16-byte unit; the
// memo's own layout is only written.  Bound by the tests' VALU work in sparse
// graphs, by the gathers in dense ones.  Against lists and pair search:
// 15 relations, C_out, 482 -> 184 us; clique of 17, PG-like, 1069 -> 603; cycle
// of 18 with 4 chords, C_out, 530 -> 332.
template <int CM>
__global__ __launch_bounds__(kBitsBlock) void k_bits_level(const DevGraph *g, uint32_t n, uint32_t k,
                                                           const Counters *cnt, BitsSpace Q, MemoPtrs M,
                                                           HeavyPart *rec, uint32_t *arrived,
                                                           unsigned long long *tally) {
    extern __shared__ __align__(16) uint32_t conn[];  // 2^n bits
    __shared__ uint32_t nb[3][256], pend[kBitsBlock / 64][128];
    __shared__ unsigned long long sums[2];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6, count = cnt->level_count[k];
    constexpr uint32_t kStride = CM == MPDP_COST_COUT ? 1u : 2u;
    const unsigned long long below = (1ull << lane) - 1ull;
    const uint32_t nw = gridDim.x * (kBitsBlock / 64), w = wave * gridDim.x + blockIdx.x;
    const uint32_t lgP = k < 7u ? k - 1u : 6u, P = 1u << lgP, sub = lane & (P - 1u), each = 64u >> lgP;
    // waves a set: as many as there are, eight rounds of candidates or more each
    uint32_t parts = 1;
    while (k >= 7u && 2u * parts * count <= min(nw, kPairWaves) && parts < 64u && (1u << (k - 7u)) >= 16u * parts)
        parts <<= 1;
    const uint32_t items = parts > 1u ? count * parts : (count + each - 1u) / each;
    if (blockIdx.x >= items) return;  // the whole workgroup
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(Q.conn);
        const uint32_t words = max(1u, (1u << n) / 128u);
        for (uint32_t i = t; i < words; i += kBitsBlock) reinterpret_cast<uint4 *>(conn)[i] = src[i];
        for (uint32_t i = t; i < 3u * 256u; i += kBitsBlock) nb[i >> 8][i & 255u] = g->lds.nb[i >> 8][i & 255u];
        if (t < 2u) sums[t] = 0ull;
    }
    const uint64_t off = g->lds.loff[k];
    const uint32_t *list = Q.list + off;
    __syncthreads();
    const auto connected = [&](uint32_t X) { return (conn[X >> 5] >> (X & 31u)) & 1u; };
    unsigned long long ccp = 0, evaluated = 0;
    for (uint32_t item = w; item < items; item += nw) {
        const uint32_t s0 = parts > 1u ? item / parts : item * each + (lane >> lgP), part = parts > 1u ? item % parts : 0u;
        const bool live = s0 < count;
        const uint32_t S = live ? list[s0] : 0u, lo = lowbit(S), rest = S ^ lo;
        const double cS = live ? Q.card[(size_t)S * kStride] : 0.0;
        SetBest best{__builtin_inf(), ~0u, ~0u};
        const auto cost_pair = [&](uint32_t A, bool on) {
            if (!on) return;
            const uint32_t B = S ^ A;
            if (CM == MPDP_COST_COUT) {
                take_best(best, pair_best<CM>(A, B, Q.cost[A], Q.cost[B], 0.0, 0.0, cS));
            } else {
                const double2 a = reinterpret_cast<const double2 *>(Q.cost)[A];
                const double2 b = reinterpret_cast<const double2 *>(Q.cost)[B];
                take_best(best, pair_best<CM>(A, B, a.x, b.x, a.y, b.y, cS));
            }
        };
        if (k < 7u) {
            const uint32_t x = deposit(sub, rest), A = lo | x;
            const bool on = live && x != rest && connected(A) && connected(S ^ A);
            ccp += on ? 1u : 0u;
            cost_pair(A, on);
        } else {
            const uint32_t rounds = (1u << (k - 7u)) / parts, step = rounds * parts > 1u ? deposit(64u, rest) : 0u;
            uint32_t x = deposit(part * rounds * 64u + lane, rest), waiting = 0;
            for (uint32_t r = 0; r < rounds; ++r) {
                const uint32_t A = lo | x;
                const bool on = x != rest && connected(A) && connected(S ^ A);
                x = ((x | ~rest) + step) & rest;  // (the masked add carries through the holes)
                ccp += on ? 1u : 0u;
                const unsigned long long m = __ballot(on);
                const uint32_t c = (uint32_t)__popcll(m);
                if (c >= 40u) {
                    cost_pair(A, on);
                } else if (c != 0u) {
                    if (on) pend[wave][waiting + (uint32_t)__popcll(m & below)] = A;
                    waiting += c;
                    wave_sync_lds();
                    if (waiting >= 64u) {
                        waiting -= 64u;
                        cost_pair(pend[wave][waiting + lane], true);
                        wave_sync_lds();
                    }
                }
            }
            cost_pair(pend[wave][lane], lane < waiting);
            wave_sync_lds();
        }
        group_best(best, P);
        // Alg. 3's candidates: a cut vertex splits S's blocks between two
        // smaller sets that share it; without one S is a block.  Lane j of the
        // set's looks at its j-th relation
        if (part == 0u) {
            const uint32_t v = sub < k ? deposit(1u << sub, S) : 0u;
            const unsigned long long cuts =
                (__ballot(live && v != 0u && !connected(S ^ v)) >> (lane & ~(P - 1u))) & (P == 64u ? ~0ull : (1ull << P) - 1ull);
            uint32_t e = (1u << k) - 2u;
            const uint32_t from = (lane & ~(P - 1u)) + (cuts ? (uint32_t)__builtin_ctzll(cuts) : 0u);
            const uint32_t cut = (uint32_t)__shfl((int)v, (int)from, 64);
            if (live && k > 2u && cuts) {
                const uint32_t R = S ^ cut;
                uint32_t seen = lowbit(R), fr = seen;
                while (fr != 0u) {
                    fr = nbrs_of<false>(nb, fr) & R & ~seen;
                    seen |= fr;
                }
                e = Q.cand[seen | cut] + Q.cand[S ^ seen];
            }
            if (live && sub == 0u) {
                Q.cand[S] = e;
                evaluated += e;
            }
        }
        bool store = live && sub == 0u;
        if (parts > 1u) store = meet_parts(PairParts{rec, arrived}, s0, part, parts, best, lane);
        if (store) {
            Q.cost[(size_t)S * kStride] = best.c;
            store_best(M, off + colex_rank(kRankTable.v, S, false),
                       Key{(unsigned long long)__double_as_longlong(best.c), best.l, best.op}, cS);
        }
    }
    for (int d = 32; d >= 1; d >>= 1) {
        ccp += (unsigned long long)__shfl_xor((long long)ccp, d);
        evaluated += (unsigned long long)__shfl_xor((long long)evaluated, d);
    }
    if (lane == 0) {
        atomicAdd(&sums[0], ccp);
        atomicAdd(&sums[1], evaluated);
    }
    __syncthreads();
    if (t < 2u) atomicAdd(&tally[2u * (blockIdx.x % kPairGrid) + t], sums[t]);
}

}  // namespace

hipError_t launch_bits_init(const DevGraph *g, uint32_t n, Counters *cnt, const BitsSpace &b, hipStream_t s) {
    hipLaunchKernelGGL(k_bits_init, dim3(((1u << n) + kBitsInitBlock - 1) / kBitsInitBlock), dim3(kBitsInitBlock), 0, s,
                       g, n, cnt, b);
    return hipGetLastError();
}

hipError_t launch_bits_level(const DevGraph *g, int cost_model, uint32_t n, uint32_t k, uint64_t sets,
                             const Counters *cnt, const BitsSpace &b, MemoPtrs memo, HeavyPart *rec, uint32_t *arrived,
                             unsigned long long *tally, hipStream_t s) {
    // waves: 64 candidates each on the lower levels, eight rounds of them from
    // nine relations on; what the bitmap leaves of the LDS is no limit
    const uint64_t lanes = sets << (k - 1);
    const uint64_t waves = std::max<uint64_t>(k < 7 ? (lanes + 63) / 64 : sets, lanes / 512);
    const uint32_t grid = (uint32_t)std::min<uint64_t>((waves + kBitsBlock / 64 - 1) / (kBitsBlock / 64), kBitsGrid);
    const uint32_t lds = std::max<uint32_t>(16u, (1u << n) / 8);
    if (cost_model == MPDP_COST_COUT)
        hipLaunchKernelGGL(k_bits_level<MPDP_COST_COUT>, dim3(grid), dim3(kBitsBlock), lds, s, g, n, k, cnt, b, memo,
                           rec, arrived, tally);
    else
        hipLaunchKernelGGL(k_bits_level<MPDP_COST_PGLIKE>, dim3(grid), dim3(kBitsBlock), lds, s, g, n, k, cnt, b, memo,
                           rec, arrived, tally);
    return hipGetLastError();
}

}  // namespace mpdp
