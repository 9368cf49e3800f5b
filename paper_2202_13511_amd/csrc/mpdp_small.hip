// A whole query of up to kSmallMaxRel relations in one launch of one
// workgroup: all 2^n memo entries live in LDS, indexed by the relation set,
// the levels are separated by workgroup barriers, and the plan goes straight
// to the caller's (pinned) memory.  One launch per level, as larger queries
// take, costs some 8 us a level before any work.
#include <hip/hip_runtime.h>

#include "mpdp_internal.h"
#include "mpdp_lists.h"

namespace mpdp {
namespace {

constexpr int kSmallBlock = 1024;
constexpr uint32_t kSmallSets = 1u << kSmallMaxRel;

struct SmallLds {
    double cost[kSmallSets], card[kSmallSets];
    uint16_t left[kSmallSets];
    uint16_t cand[kSmallSets];      // Alg. 3 candidates of the set (sum over its blocks of 2^b - 2)
    uint16_t list[kSmallSets];      // connected sets, level k from loff[k]
    uint8_t op[kSmallSets];
    uint32_t conn[kSmallSets / 32]; // bit S: S is connected
    uint32_t nb[2][64], ch[2][64];  // neighbours / children of a set, by its low and high six relations
    uint2 pd[16];
    uint32_t count[16], loff[16];
    uint32_t node_set[2 * kSmallMaxRel], node_at[2 * kSmallMaxRel];  // a plan node's set, joins finished before it
    uint32_t q_set[16], q_start[16];
    unsigned long long ccp, evaluated;
    int error;
};

__device__ __forceinline__ bool small_conn(const SmallLds &D, uint32_t S) { return (D.conn[S >> 5] >> (S & 31u)) & 1u; }

__device__ __forceinline__ uint32_t small_grow(const SmallLds &D, uint32_t seed, uint32_t R) {
    uint32_t seen = seed, fr = seed;
    while (fr) {
        fr = (D.nb[0][fr & 63u] | D.nb[1][fr >> 6]) & R & ~seen;
        seen |= fr;
    }
    return seen;
}

// Alg. 3 candidates of a connected set: a cut vertex splits its blocks
// between two smaller sets that share it; without one the set is a block.
__device__ __forceinline__ uint32_t small_candidates(const SmallLds &D, uint32_t S, uint32_t k) {
    uint32_t cut = 0;
#pragma unroll
    for (uint32_t v = 0; v < kSmallMaxRel; ++v) {
        const uint32_t R = S & ~(1u << v);  // (itself, where v is not a member)
        cut |= small_conn(D, R) ? 0u : 1u << v;
    }
    if (k == 2u || cut == 0u) return (1u << k) - 2u;
    const uint32_t v = lowbit(cut), part = small_grow(D, lowbit(S ^ v), S ^ v);
    return (uint32_t)D.cand[part | v] + D.cand[S ^ part];
}

// The pairs (A[j], S - A[j]) with on[j], both orientations, without branches.
template <int CM, int R>
__device__ __forceinline__ void small_offers(const SmallLds &D, uint32_t S, const uint32_t *A, const bool *on,
                                             double cS, SetBest &best) {
    double cA[R], cB[R], kA[R], kB[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        cA[j] = D.cost[A[j]];
        cB[j] = D.cost[S ^ A[j]];
        kA[j] = CM == MPDP_COST_COUT ? 0.0 : D.card[A[j]];
        kB[j] = CM == MPDP_COST_COUT ? 0.0 : D.card[S ^ A[j]];
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
        SetBest o = pair_best<CM>(A[j], S ^ A[j], cA[j], cB[j], kA[j], kB[j], cS);
        o.l = on[j] ? o.l : ~0u;
        o.c = on[j] ? o.c : __builtin_inf();
        take_best(best, o);
    }
}

// The workgroup's 16 waves:
//  1. every subset's card and connectivity, the connected ones into their
//     level's list.  A lane's subsets t, t + 1024, .. differ in relations 10
//     and 11 alone, so they share the product over the lower ones; a member
//     outside the subset multiplies by an exact 1.0;
//  2. level by level, each connected set by 1 to 64 lanes (as many as the
//     level's sets leave): a tree join's pairs are its edges (Alg. 2);
//     otherwise every subset that holds the lowest relation, kept when both
//     sides are connected (bit lookups), while the upper four waves count
//     Alg. 3's candidates;
//  3. the plan by wave 0, the memo by the others.
// Bound by latency: some 5 k cycles a level of LDS round trips and a barrier,
// 27 us for star 12, C_out.  The whole call took 95 us in 13 launches and two
// copies and takes 40; 9 relations with extra predicates, PG-like, took 288 us
// (34 launches) and take 45.
template <int CM>
__global__ __launch_bounds__(kSmallBlock) void k_small(SmallQuery Q, MemoPtrs M, SmallOut *out) {
    __shared__ SmallLds D;
    const uint32_t t = threadIdx.x, lane = t & 63u, n = Q.n, N = 1u << n;
    const unsigned long long below = (1ull << lane) - 1ull;
    if (t < 128u) {
        const uint32_t x = t & 63u, shift = t < 64u ? 0u : 6u;
        uint32_t a = 0, c = 0;
#pragma unroll
        for (uint32_t b = 0; b < 6u; ++b) {
            const uint32_t av = shift ? Q.adj[6 + b] : Q.adj[b], cv = shift ? Q.kids[6 + b] : Q.kids[b];
            a |= ((x >> b) & 1u) ? av : 0u;
            c |= ((x >> b) & 1u) ? cv : 0u;
        }
        D.nb[shift ? 1 : 0][x] = a;
        D.ch[shift ? 1 : 0][x] = c;
    } else if (t < 144u) {
        D.count[t - 128u] = 0;
        D.loff[t - 128u] = Q.loff[t - 128u];
        if (t == 128u) {
            D.ccp = 0;
            D.evaluated = 0;
            D.error = 0;
        }
    } else if (t >= 192u && t - 192u < n) {
        const uint32_t v = t - 192u;
        D.pd[v] = make_uint2(Q.pd[v][0], Q.pd[v][1]);
        D.cost[1u << v] = Q.bcost[v];
        D.left[1u << v] = 0;
        D.op[1u << v] = MPDP_OP_SCAN;
        D.cand[1u << v] = 0;
    }
    __syncthreads();

    double low = 1.0;  // product over relations 0 .. 9
#pragma unroll
    for (uint32_t v = 0; v < 10u; ++v)
        if (v < n) {
            const bool has = (t >> v) & 1u;
            low = low * (has ? Q.card[v] : 1.0);
            const uint32_t av = Q.adj[v];
#pragma unroll
            for (uint32_t u = 0; u < v; ++u)
                if ((av >> u) & 1u) low = low * (has && ((t >> u) & 1u) ? Q.sel[v * (v - 1u) / 2u + u] : 1.0);
        }
    // lanes with as many bits in their number as this lane's, and (lanes 0 ..
    // 6) lanes with `lane` bits
    const uint32_t pl = (uint32_t)popc32(lane);
    unsigned long long like_me = 0, of_pop = 0;
#pragma unroll
    for (uint32_t j = 0; j < 7u; ++j) {
        const unsigned long long m = __ballot(pl == j);
        like_me = pl == j ? m : like_me;
        of_pop = lane == j ? m : of_pop;
    }
    for (uint32_t S0 = 0; S0 < N; S0 += kSmallBlock) {
        const uint32_t S = S0 + t;
        const uint32_t k = (uint32_t)popc32(S);
        const bool in = S < N;
        double c = low;
#pragma unroll
        for (uint32_t v = 10u; v < kSmallMaxRel; ++v)
            if ((S0 >> v) & 1u) {
                c = c * Q.card[v];
                for (uint32_t U = Q.adj[v] & ((1u << v) - 1u); U; U &= U - 1u) {
                    const uint32_t u = (uint32_t)ctz32(U);
                    c = c * ((S >> u) & 1u ? Q.sel[v * (v - 1u) / 2u + u] : 1.0);
                }
            }
        bool conn = false;
        if (in && S != 0u) {
            if (Q.is_tree)  // a forest of k - 1 edges is one tree
                conn = (uint32_t)popc32(S & (D.ch[0][S & 63u] | D.ch[1][S >> 6])) == k - 1u;
            else
                conn = small_grow(D, lowbit(S), S) == S;
        }
        if (in) D.card[S] = c < 1.0 ? 1.0 : c;
        const unsigned long long cm = __ballot(conn);
        if (in && (lane & 31u) == 0u) D.conn[S >> 5] = (uint32_t)(cm >> lane);
        // the wave's sets of each level: its lanes' sets hold `high` relations
        // above the lane's own bits; one atomic, lane j for j of those
        const uint32_t high = k - pl;
        const uint32_t mine = lane < 7u && high + lane >= 2u ? (uint32_t)__popcll(cm & of_pop) : 0u;
        uint32_t at = 0;
        if (mine) at = atomicAdd(&D.count[high + lane], mine);
        at = (uint32_t)__shfl((int)at, (int)pl) + (uint32_t)__popcll(cm & like_me & below);
        if (conn && k >= 2u) D.list[D.loff[k] + at] = (uint16_t)S;
    }
    __syncthreads();

    unsigned long long ccp = 0, evaluated = 0;
    const uint32_t threads = Q.is_tree ? kSmallBlock : kSmallBlock - 256;  // that cost pairs
    for (uint32_t k = 2; k <= n; ++k) {
        const uint32_t count = D.count[k], cands = Q.is_tree ? n - 1u : (1u << (k - 1u)) - 1u;
        if (t >= threads) {
            for (uint32_t i = t - threads; i < count; i += kSmallBlock - threads) {
                const uint32_t S = D.list[D.loff[k] + i], e = small_candidates(D, S, k);
                D.cand[S] = (uint16_t)e;
                evaluated += e;
            }
            __syncthreads();
            continue;
        }
        uint32_t lgP = 0;
        while (lgP < 6u && (2u * count << lgP) <= threads && (2u << lgP) <= cands + 1u) ++lgP;
        const uint32_t P = 1u << lgP, sub = t & (P - 1u);
        for (uint32_t i = t >> lgP; i < count; i += threads >> lgP) {
            const uint32_t S = D.list[D.loff[k] + i];
            const double cS = D.card[S];
            SetBest best{__builtin_inf(), ~0u, ~0u};
            if (Q.is_tree) {
                for (uint32_t v0 = sub; v0 < n; v0 += 4u << lgP) {
                    // four members' pairs, their reads in flight together (a
                    // member without one reads its own entry)
                    uint32_t A[4];
                    bool on[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t v = v0 + ((uint32_t)j << lgP);
                        const uint2 pd = D.pd[v & 15u];
                        on[j] = v < n && ((S >> v) & 1u) && (S & pd.x);
                        A[j] = on[j] ? pd.y & S : lowbit(S);
                        ccp += on[j] ? 1u : 0u;
                    }
                    small_offers<CM, 4>(D, S, A, on, cS, best);
                }
                evaluated += sub == 0u ? 2ull * (k - 1u) : 0ull;
            } else {
                // the sub-th subset of S without its lowest relation, then
                // every P-th (a masked add carries through the holes)
                const uint32_t lo = lowbit(S), rest = S ^ lo;
                const uint32_t step = P < (1u << (k - 1u)) ? deposit(P, rest) : 0u;
                uint32_t x = deposit(sub, rest);
                for (uint32_t j = sub; j < cands; j += 2u * P) {
                    uint32_t A[2];
                    bool on[2];
                    A[0] = lo | x;
                    x = ((x | ~rest) + step) & rest;
                    A[1] = lo | x;
                    x = ((x | ~rest) + step) & rest;
                    on[0] = small_conn(D, A[0]) & small_conn(D, S ^ A[0]);
                    on[1] = (j + P < cands) & small_conn(D, A[1]) & small_conn(D, S ^ A[1]);
                    ccp += (on[0] ? 1u : 0u) + (on[1] ? 1u : 0u);
                    if (on[0] | on[1]) small_offers<CM, 2>(D, S, A, on, cS, best);
                }
            }
            group_best(best, P);
            if (sub == 0u) {
                D.cost[S] = best.c;
                D.left[S] = (uint16_t)best.l;
                D.op[S] = (uint8_t)best.op;
            }
        }
        __syncthreads();
    }
    for (int off = 32; off >= 1; off >>= 1) {
        ccp += (unsigned long long)__shfl_xor((long long)ccp, off);
        evaluated += (unsigned long long)__shfl_xor((long long)evaluated, off);
    }
    if (lane == 0) {
        atomicAdd(&D.ccp, ccp);
        atomicAdd(&D.evaluated, evaluated);
    }

    // the memo entries of the connected sets (waves 1 ..), if there is a memo
    if (t >= 64u && M.cost) {
        for (uint32_t S = t - 64u; S < N; S += kSmallBlock - 64u) {
            if (!((D.conn[S >> 5] >> (S & 31u)) & 1u)) continue;
            const uint32_t c6 = (uint32_t)popc32(S & 63u);
            const uint32_t at = D.loff[popc32(S)] + kRankTable.v[S & 63u] + kRankTable.v[64 + (c6 << 6) + (S >> 6)];
            M.cost[at] = D.cost[S];
            M.card[at] = D.card[S];
            M.left[at] = D.left[S];
            M.op[at] = D.op[S];
        }
    }
    // the plan (wave 0): join nodes are numbered in post-order after the n
    // relations, so a node's number follows from the sizes alone (see
    // extract_plan).  One round per depth finds every node's inputs; a lane
    // goes on with one joined input itself and passes a second one on.
    if (t < 64u) {
        uint32_t S = t == 0 ? N - 1u : 0u, start = 0;
        bool bad = false;
        for (uint32_t depth = 0; depth < n && __ballot(S != 0u) != 0ull; ++depth) {
            uint32_t c1 = 0, s1 = 0;
            if (S) {
                const uint32_t Lf = D.left[S], Rt = S ^ Lf;
                if (Lf == 0u || (Lf & ~S) != 0u || Rt == 0u) {
                    bad = true;
                    S = 0;
                } else {
                    const uint32_t nl = (uint32_t)popc32(Lf), nr = (uint32_t)popc32(Rt), rs = start + nl - 1u;
                    D.node_set[n + start + nl + nr - 2u] = S;
                    D.node_at[n + start + nl + nr - 2u] = start;
                    if (nl >= 2u && nr >= 2u) { c1 = Rt; s1 = rs; }
                    start = nl >= 2u ? start : rs;
                    S = nl >= 2u ? Lf : (nr >= 2u ? Rt : 0u);
                }
            }
            const unsigned long long m = __ballot(c1 != 0u);
            if (m != 0ull) {  // at most n / 2 joins at one depth
                const uint32_t at = (uint32_t)__popcll(m & below);
                if (c1) {
                    D.q_set[at & 15u] = c1;
                    D.q_start[at & 15u] = s1;
                }
                wave_sync_lds();
                const unsigned long long idle = __ballot(S == 0u);
                const uint32_t r = (uint32_t)__popcll(idle & below);
                if (S == 0u && r < (uint32_t)__popcll(m)) {
                    S = D.q_set[r & 15u];
                    start = D.q_start[r & 15u];
                }
                wave_sync_lds();
            }
        }
        if (__ballot(bad || S != 0u) != 0ull && lane == 0) D.error = 1;
        wave_sync_lds();
        if (D.error == 0 && t < 2u * n - 1u) {
            const uint32_t set = t < n ? 1u << t : D.node_set[t];
            mpdp_plan_node p;
            p.left = p.right = -1;
            if (t >= n) {
                const uint32_t Lf = D.left[set], Rt = set ^ Lf, at = D.node_at[t];
                const uint32_t nl = (uint32_t)popc32(Lf), nr = (uint32_t)popc32(Rt);
                p.left = nl >= 2u ? (int)(n + at + nl - 2u) : ctz32(Lf);
                p.right = nr >= 2u ? (int)(n + at + nl + nr - 3u) : ctz32(Rt);
            }
            p.relset = set;
            p.op = D.op[set];
            p.cost = D.cost[set];
            p.card = D.card[set];
            out->plan[t] = p;
        }
    }
    __syncthreads();
    if (t == 0) {
        uint32_t sets = 0;
        for (uint32_t k = 2; k <= n; ++k) sets += D.count[k];
        out->root = D.cost[N - 1u];
        out->connected = sets;
        out->ccp = D.ccp;
        out->evaluated = D.evaluated;
        out->error = (uint32_t)D.error;
    }
}

}  // namespace

hipError_t launch_small(const SmallQuery &q, int cost_model, MemoPtrs memo, SmallOut *out, hipStream_t s) {
    if (cost_model == MPDP_COST_COUT)
        hipLaunchKernelGGL(k_small<MPDP_COST_COUT>, dim3(1), dim3(kSmallBlock), 0, s, q, memo, out);
    else
        hipLaunchKernelGGL(k_small<MPDP_COST_PGLIKE>, dim3(1), dim3(kSmallBlock), 0, s, q, memo, out);
    return hipGetLastError();
}

}  // namespace mpdp
