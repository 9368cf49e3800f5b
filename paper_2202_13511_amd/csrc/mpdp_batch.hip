// Batched optimization of many small queries in one persistent launch.
//
// Each workgroup pulls the next query from an atomic counter and runs the
// whole level loop of Alg. 5 for it, with workgroup barriers between levels
// instead of kernel launches: it builds the query's LDS image from the raw
// edges, cardinalities and selectivities, fills the base relations, runs
// levels 2..n, rebuilds the plan and records the device wall clock at the
// query's start and end.  A level is its list of connected sets, grown from
// the level before (see mpdp_lists.h): tree joins cost their edges (Alg. 2),
// the others search their csg-cmp pairs or, in dense graphs, walk the subsets
// of their sets; of a star around relation 0 every set of relation 0 and
// others is connected, so it needs no lists, and trees of many connected sets
// are unranked.  Memo and scratch live in a per-workgroup slot that is reused
// from query to query, so the workspace does not grow with the batch.  A large
// query may be taken by a team of workgroups (consecutive queue entries): they
// split the sets of every level and meet at barriers, in the slot of the team's
// first member.  Entries are taken in queue order within their share, so of
// each share at most one team waits for members, for kTeamFormTicks at most:
// those that have come by then are the team, and a workgroup that takes an entry
// of it later passes it by.  So a launch ends however few of its workgroups the
// device runs at a time.
#include <hip/hip_runtime.h>

#include "mpdp_device.h"
#include "mpdp_internal.h"
#include "mpdp_lists.h"

namespace mpdp {
namespace {

constexpr int kBatchBlock = 512;
constexpr int kBW = kBatchBlock / 64;
// members per gather batch of an unranked tree set: three keeps the kernel
// (every path of a query inlined, 128 registers per lane) from more spilling
constexpr int kBatchPairBatch = 3;
constexpr unsigned long long kTeamWaitTicks = 200000000ull;  // 2 s of the 100 MHz device clock
// 2 ms: longer than the members of a team take to come where the device has
// room for them (0.5, 2 and 10 ms give the same times on batches of all sizes),
// and little to wait for each team where it has not
constexpr unsigned long long kTeamFormTicks = 200000ull;

__device__ __forceinline__ uint32_t load_shared_count(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The workgroups of a team meet here for the `phase`-th time.  Every wave
// first waits until its own stores (memo, lists) have reached the L2; then
// one thread per workgroup arrives, and after the wait drops the lines other
// members may have written from this CU's cache (agent-scope acquire), once
// for all its waves.  `spread`: the members run on several XCDs, so the
// thread writes the L2 back before it arrives (agent-scope release).  That
// takes some 40 us with hundreds of workgroups at work, and members of one
// XCD, which share its L2, don't need it.  The
// wait is bounded by the device clock: past kTeamWaitTicks the team is marked
// failed, and every later wait of that team returns at once.  Returns false
// once the team has failed; its members then leave the query (its lists may
// be incomplete), and the query reports an error.
__device__ bool team_barrier(TeamRec *R, uint32_t team, bool spread, uint32_t &phase, uint32_t &s_ok) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (spread) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __hip_atomic_fetch_add(&R->arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t target = team * (phase + 1u);
        const unsigned long long start = wall_clock64();
        while (__hip_atomic_load(&R->arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target &&
               __hip_atomic_load(&R->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) {
            __builtin_amdgcn_s_sleep(2);
            if ((unsigned long long)wall_clock64() - start > kTeamWaitTicks) {
                __hip_atomic_store(&R->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
        }
        s_ok = __hip_atomic_load(&R->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    ++phase;
    __syncthreads();
    return s_ok != 0u;
}

// This workgroup's place in the team (kTeamClosed set: it came too late).  Its
// XCD is in the record before it counts.  One thread.
__device__ __forceinline__ uint32_t join_team(TeamRec *R, uint32_t xcd) {
    __hip_atomic_fetch_or(&R->xcds, 1u << xcd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    return __hip_atomic_fetch_add(&R->joined, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The team is formed: its leader (member 0), whose memo slot is set up, closes
// it when `most` workgroups have joined or kTeamFormTicks have passed, and
// publishes slot and size; the others wait for that, and see the slot's
// contents afterwards.  Returns TeamRec::formed, 0 if it did not come (the wait
// is bounded; the leader's is shorter).
__device__ uint32_t form_team(TeamRec *R, uint32_t most, uint32_t member, uint32_t slot, uint32_t &s_ok) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long start = wall_clock64();
        uint32_t formed;
        if (member == 0u) {
            while (load_shared_count(&R->joined) < most && (unsigned long long)wall_clock64() - start < kTeamFormTicks)
                __builtin_amdgcn_s_sleep(2);
            formed = __hip_atomic_fetch_or(&R->joined, kTeamClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t xcds = load_shared_count(&R->xcds);
            if (xcds & (xcds - 1u)) {
                formed |= kTeamSpread;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            }
            __hip_atomic_store(&R->slot, slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_s_waitcnt(0);
            __hip_atomic_store(&R->formed, formed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            while ((formed = load_shared_count(&R->formed)) == 0u) {
                __builtin_amdgcn_s_sleep(2);
                if ((unsigned long long)wall_clock64() - start > kTeamWaitTicks) {
                    __hip_atomic_store(&R->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        s_ok = formed;
    }
    __syncthreads();
    return s_ok;
}

// The XCD this workgroup runs on (hardware register XCC_ID).
__device__ __forceinline__ uint32_t xcd_id() { return (uint32_t)__builtin_amdgcn_s_getreg(20 | (3 << 11)) & 7u; }

// The next queue entry: of the XCD's own share, of the common rest, of the
// other shares; bc->entries when there is none.  `end`: share_end.  A batch
// without teams has no shares and reads no counter but `next` (with every
// workgroup looking through the shares as it came and went, 500 queries of
// two relations took 106 us; they take 30).  One thread.
__device__ uint32_t take_entry(BatchCounters *bc, const uint32_t *end, uint32_t entries, uint32_t xcd, bool &own) {
    for (uint32_t y = 0; y < 9u; ++y) {
        if (y == 1u) {  // after the own share
            own = false;
            const uint32_t i = atomicAdd(&bc->next, 1u);
            if (i < entries) return i;
        }
        if ((y == 0u && !own) || end[7] == 0u) continue;
        const uint32_t x = (xcd + y) & 7u;
        const uint32_t first = x ? end[x - 1u] : 0u;
        if (end[x] == first || load_shared_count(&bc->share_taken[x]) >= end[x] - first) continue;
        const uint32_t i = first + atomicAdd(&bc->share_taken[x], 1u);
        if (i < end[x]) return i;
    }
    return entries;
}


// Workgroups' LDS, two per CU: 160 KB / 2 less the image.  A search path
// leaves less than two states per relation behind.
constexpr uint32_t kBatchPool = 240;
using BatchBuf = PairBufN<kBatchPool, 2 * kBatchMaxRel>;
static_assert(3 * (kBatchPool + 2 * kBatchMaxRel) >= 64 * (kBatchMaxRel / 2), "block_candidates' pieces");

// What the waves keep while a level runs; the plan is rebuilt in its place.
union BatchScratch {
    BatchBuf pairs[kBW];
    struct {
        uint32_t set[kBW][flat_block_words(kTreeChunkMax)], bsum[kBW][flat_block_words(kTreeChunkMax)];
    } flat;
    struct {
        uint32_t set[kBW][tree_ring(4, 1)], bsum[kBW][tree_ring(4, 1)];
    } ring;
    uint32_t grow[sizeof(BatchBuf) * kBW / 4];  // expand_sets, expand_tree
    PlanScratch plan;
};

// Build the LDS image of one query inside the workgroup (everything except
// the binomials, which are staged once per workgroup; no children table).
// num, kids: scratch, a tree join's preorder numbers and children in them.
__device__ void build_image(LdsGraph &L, const BatchQueryDev &Q, const uint32_t *edges, const double *cards,
                            const double *sels, const double *bcosts, uint32_t *num, uint32_t *kids) {
    const uint32_t t = threadIdx.x, n = Q.n, m = Q.m, full = (1u << n) - 1u;
    const uint32_t *E = edges + 2ull * Q.edge_off;
    const double *C = cards + Q.card_off;
    const double *SL = sels + Q.edge_off;
    if (t < kMaxRel) {
        L.adj[t] = 0;
        L.pd[t][0] = 0;
        L.lo[t][0] = 0;
        L.lo[t][1] = 0;
        L.csel[t][0] = t < n ? C[t] : 1.0;
        L.csel[t][1] = 1.0;
        L.pd[t][1] = 1u << t;
        L.card[t] = t < n ? C[t] : 1.0;
        if (t >= n) L.bcost[t] = 0.0;
        else if (bcosts) L.bcost[t] = bcosts[Q.card_off + t];  // planned intermediate results
        else L.bcost[t] = Q.cost_model == MPDP_COST_PGLIKE ? 0.01 * C[t] : 0.0;
    } else if (t >= 64u && t < 98u) {
        const uint32_t k = t - 64u;
        uint64_t off = 0;
        for (uint32_t j = 0; j < k && j <= n; ++j) off += L.binom[n * 33 + j];
        L.loff[k] = off;
    }
    __syncthreads();
    for (uint32_t e = t; e < m; e += blockDim.x) {
        const uint32_t u = E[2 * e], v = E[2 * e + 1];
        atomicOr(&L.adj[u], 1u << v);
        atomicOr(&L.adj[v], 1u << u);
    }
    __syncthreads();
    if (t < 64u) {  // wave 0
        // selectivities of edges (u, v), u < v, grouped by v, u ascending
        const uint32_t lower = t < n ? L.adj[t] & ((1u << t) - 1u) : 0u;
        uint32_t start = 0;
        for (uint32_t w = 0; w < n; ++w) start += w < t ? (uint32_t)popc32(L.adj[w] & ((1u << w) - 1u)) : 0u;
        if (t < n) {
            L.selrow[t] = start;
            L.lo[t][0] = lowbit(lower);
            L.lo[t][1] = lower & ~lowbit(lower);
        }
        wave_sync_lds();
        for (uint32_t e = t; e < m; e += 64u) {
            const uint32_t a = E[2 * e], b = E[2 * e + 1];
            const uint32_t hi = a > b ? a : b, lo = a > b ? b : a;
            L.sel[L.selrow[hi] + (uint32_t)popc32(L.adj[hi] & ((1u << lo) - 1u))] = SL[e];
        }
        wave_sync_lds();
        if (lower) L.csel[t][1] = L.sel[start];
    } else if (t < 128u && Q.is_tree) {  // wave 1, relation v = lane
        // rooted at relation 0: parents by breadth-first rounds, subtrees from
        // the last round up, preorder numbers from the first down
        const uint32_t v = t - 64u, av = v < n ? L.adj[v] : 0u;
        uint32_t fr = 1u, seen = 1u, depth = 0, round = 0, par = 0;
        while (seen != full) {
            ++round;
            const bool in = (av & fr) != 0u && ((seen >> (v & 31u)) & 1u) == 0u;
            if (in) {
                par = av & fr;
                depth = round;
            }
            fr = (uint32_t)__ballot(in);
            if (fr == 0u) break;
            seen |= fr;
        }
        const uint32_t last = round, up = par ? (uint32_t)ctz32(par) : 0u;
        if (v < n) L.pd[v][0] = par;
        for (uint32_t d = last; d >= 1u; --d) {
            wave_sync_lds();
            if (depth == d && par) atomicOr(&L.pd[up][1], L.pd[v][1]);
        }
        wave_sync_lds();
        if (v < n) kids[v] = 0;
        uint32_t before = 1;  // relations between the parent and v in preorder, and the parent
        if (par)
            for (uint32_t U = L.adj[up] & ~L.pd[up][0] & ((1u << v) - 1u); U; U &= U - 1u)
                before += (uint32_t)popc32(L.pd[ctz32(U)][1]);
        if (v == 0u) num[0] = 0;
        for (uint32_t d = 1; d <= last; ++d) {
            wave_sync_lds();
            if (depth == d && par) num[v] = num[up] + before;
        }
        wave_sync_lds();
        if (par) atomicOr(&kids[num[up]], 1u << num[v]);
    }
    __syncthreads();
    // tables by bitmap byte (only those that n relations reach): neighbours of
    // a set; children and own numbers of a set in preorder numbers
    const uint32_t bytes = (n + 7u) / 8u;
    for (uint32_t i = t; i < 4u * 256u; i += blockDim.x) {
        const uint32_t byte = i >> 8, x = i & 255u;
        if (byte >= bytes && x != 0u) continue;
        uint32_t a = 0, c = 0, p = 0;
        if (!Q.is_tree) {
            for (uint32_t j = 0; j < 8u; ++j) a |= ((x >> j) & 1u) && 8u * byte + j < n ? L.adj[8u * byte + j] : 0u;
            L.nb[byte][x] = a;
        } else {
            for (uint32_t v = 0; v < n; ++v) {
                const uint32_t at = num[v];
                if ((at >> 3) == byte && ((x >> (at & 7u)) & 1u)) {
                    c |= kids[at];
                    p |= 1u << v;
                }
            }
            L.pch[byte][x] = c;
            L.perm[byte][x] = p;
            if (Q.sched & kSchedUnrank) {
                uint32_t own = 0;  // children in the query's own numbers
                for (uint32_t v = 1; v < n; ++v) own |= (L.pd[v][0] & (x << (8u * byte))) ? 1u << v : 0u;
                L.ch[byte][x] = own;
            }
        }
    }
    __syncthreads();
}

// Least sets that a wave takes at a time on a cyclic query's level: a wave of
// fewer has too few search states, while other queries wait for the CU
// (4096 queries: 7.78 ms with 1, 7.64 with 16, 7.70 with 32).
constexpr uint32_t kBatchPer = 16;

// Two workgroups a CU: 16 waves, 128 registers a lane (some 50 spilled, in the
// set-up and the plan).  4096 mixed queries of 8-20 relations, C_out, took
// 14.7 ms while every level unranked and tested all C(n, k) subsets and every
// block's subsets were walked, and take 4.8; per query on one workgroup a
// chain of 20 went from 1.42 to 0.16 ms, a cycle of 20 with up to two chords
// from 2.89 to 0.87, a 20-relation tree with one to three extra edges from
// more than 3.4 to 1.15.
template <int CM>
__global__ __launch_bounds__(kBatchBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_batch(const BatchQueryDev *qs, const uint32_t *edges,
                                                       const double *cards, const double *sels,
                                                       const double *bcosts, const uint32_t *binom_g, char *slots, uint64_t slot_bytes,
                                                       uint32_t maxn, mpdp_plan_node *plans, BatchOut *out,
                                                       TeamRec *teams, BatchCounters *bc) {
    __shared__ __align__(16) LdsGraph L;
    __shared__ __align__(16) uint32_t ranks[kRankWords24];
    __shared__ __align__(16) BatchScratch W;
    __shared__ __align__(16) HeavyPart parts_rec[kBW];
    __shared__ uint32_t parts_arrived[kBW];
    __shared__ ExpandEnds ends;
    __shared__ uint32_t s_q, s_ok, s_end[8];  // (s_end: by wave 0 alone)
    __shared__ uint32_t s_count[24];  // connected sets per level k
    __shared__ uint32_t s_num[kMaxRel], s_kids[kMaxRel];
    __shared__ unsigned long long s_conn, s_ccp, s_eval, s_t0;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    if (t == 0) atomicMin(&bc->t0, (unsigned long long)wall_clock64());
    // the entry count travels with the uploaded data, so a recorded launch
    // serves any run with the same layout
    const uint32_t nq = bc->entries;
    if (t < 8) s_end[t] = bc->share_end[t];
    for (uint32_t i = t; i < 33 * 33; i += blockDim.x) L.binom[i] = binom_g[i];
    stage_ranks(ranks, kBatchMaxRel);
    if (t < kBW) parts_arrived[t] = 0;

    // a workgroup's slot: memo (cost, card, left, op over 2^maxn entries, a
    // set's entry at the set itself, or, of a tree join, whose many sets are
    // then neighbours, at its level and rank), two set lists
    // of cap entries (level k uses list k mod 2), and a team's shared sets
    const uint64_t N = 1ull << maxn;
    const uint64_t list_off = (21 * N + 255) & ~255ull;
    // sets of the widest level; read from global memory: the LDS copy of the
    // table is complete only after the first barrier below
    const uint32_t cap = binom_g[maxn * 33 + maxn / 2];

    const uint32_t xcd = xcd_id();
    bool own = true;
    if (t < 64u) wave_sync_lds();
    for (;;) {
        if (t == 0) s_q = take_entry(bc, s_end, nq, xcd, own);
        __syncthreads();
        const uint32_t q = s_q;
        if (q >= nq) break;
        const BatchQueryDev Q = qs[q];
        const bool team = Q.team > 1;
        TeamRec *R = team ? teams + Q.team_rec : nullptr;
        uint32_t phase = 0;
        build_image(L, Q, edges, cards, sels, bcosts, s_num, s_kids);
        const uint32_t n = Q.n;
        const bool star = Q.is_tree && L.adj[0] == (1u << n) - 2u;
        const bool unrank = (Q.sched & kSchedUnrank) != 0u, walk = (Q.sched & kSchedWalk) != 0u;
        if (t == 0) {
            s_t0 = (unsigned long long)wall_clock64();
            s_conn = 0;
            s_ccp = 0;
            s_eval = 0;
        }
        // a team works in its first member's slot, published through the team record
        uint32_t slot_id = blockIdx.x, member = 0, size = 1;
        if (team) {
            if (t == 0) s_q = join_team(R, xcd);
            __syncthreads();
            member = s_q;
            if (member & kTeamClosed) {  // too late
                __syncthreads();
                continue;
            }
        }
        char *slot = slots + (uint64_t)slot_id * slot_bytes;
        MemoPtrs M{reinterpret_cast<double *>(slot), reinterpret_cast<double *>(slot + 8 * N),
                   reinterpret_cast<uint32_t *>(slot + 16 * N), reinterpret_cast<uint8_t *>(slot + 20 * N)};
        uint32_t *even = reinterpret_cast<uint32_t *>(slot + list_off), *odd = even + cap;
        const uint64_t parts_off = (list_off + 8ull * cap + 15) & ~15ull;
        if (t < 24) s_count[t] = t == 2u ? Q.m : 0u;
        if (member == 0) {
            if (t < n) {
                const uint64_t at = Q.is_tree ? L.loff[1] + t : 1u << t;
                M.cost[at] = L.bcost[t];
                M.card[at] = L.card[t];
                M.left[at] = 0;
                M.op[at] = MPDP_OP_SCAN;
            }
            // the sets of two relations: the edges
            if (Q.is_tree) {
                if (t < n) first_tree_list(L, t, even);
            } else {
                for (uint32_t e = t; e < Q.m; e += blockDim.x)
                    even[e] = (1u << edges[2ull * (Q.edge_off + e)]) | (1u << edges[2ull * (Q.edge_off + e) + 1]);
            }
            if (team) {
                if (t < kTeamSize * kBW) reinterpret_cast<uint32_t *>(slot + parts_off + sizeof(HeavyPart) * kTeamSize * kBW)[t] = 0;
                if (t == 0) __hip_atomic_store(&R->count[2], Q.m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        bool failed = false, spread = false;
        if (team) {
            const uint32_t formed = form_team(R, Q.team, member, slot_id, s_ok);
            failed = formed == 0u;
            spread = (formed & kTeamSpread) != 0u;
            size = formed & ~kTeamSpread;
            slot_id = load_shared_count(&R->slot);
            slot = slots + (uint64_t)slot_id * slot_bytes;
            M = MemoPtrs{reinterpret_cast<double *>(slot), reinterpret_cast<double *>(slot + 8 * N),
                         reinterpret_cast<uint32_t *>(slot + 16 * N), reinterpret_cast<uint8_t *>(slot + 20 * N)};
            even = reinterpret_cast<uint32_t *>(slot + list_off);
            odd = even + cap;
        } else {
            __syncthreads();
        }
        if (walk && !failed) {  // no plan yet for sets of two or more relations (base relations: the first member)
            for (uint32_t S = member * kBatchBlock + t; S < (1u << n); S += size * kBatchBlock)
                if ((S & (S - 1u)) != 0u || S == 0u) M.cost[S] = -1.0;
            if (team) failed = !team_barrier(R, size, spread, phase, s_ok);
            else __syncthreads();
        }
        // (a record and a counter for each of the team's waves: a team has
        // kTeamMinRel relations or more, and its slot room for a third list)
        const PairParts pp = team ? PairParts{reinterpret_cast<HeavyPart *>(slot + parts_off),
                                              reinterpret_cast<uint32_t *>(slot + parts_off + sizeof(HeavyPart) * kTeamSize * kBW)}
                                  : PairParts{parts_rec, parts_arrived};
        // this workgroup's waves among the team's, neighbours in other members
        const uint32_t nw = size * kBW, w = wave * size + member;
        uint32_t *counts = team ? R->count : s_count;
        unsigned long long my_sets = 0, my_ccp = 0, my_eval = 0;
        for (uint32_t k = 2; k <= n && !failed; ++k) {
            const uint32_t *list = (k & 1u) ? odd : even;
            uint32_t *next = (k & 1u) ? even : odd;
            const uint32_t count = star ? L.binom[(n - 1) * 33 + k - 1] : unrank ? 0u : team ? load_shared_count(&counts[k]) : counts[k];
            if (star) {
                constexpr int kR = flat_sets_per_lane<CM>();
                switch (Q.sched & kSchedChunkMask) {  // consecutive ranks per lane
                    case 0:
                        level_flat_wave<CM, 1, 1>(L, M, (int)n, k, 0, count, w, nw, W.flat.set[wave], W.flat.bsum[wave], lane);
                        break;
                    case 1:
                        level_flat_wave<CM, 2, kR>(L, M, (int)n, k, 0, count, w, nw, W.flat.set[wave], W.flat.bsum[wave], lane);
                        break;
                    default:
                        level_flat_wave<CM, 4, kR>(L, M, (int)n, k, 0, count, w, nw, W.flat.set[wave], W.flat.bsum[wave], lane);
                        break;
                }
            } else if (unrank) {
                const uint32_t subsets = L.binom[n * 33 + k];
                const uint32_t found = level_tree_wave<CM, 4, 1, true, false, false, kBatchPairBatch>(
                    L, M, (int)n, k, subsets, w, nw, (subsets + 255u) / 256u, W.ring.set[wave], W.ring.bsum[wave], lane);
                if (lane == 0) {
                    my_sets += found;
                    my_ccp += (unsigned long long)(k - 1) * found;
                    my_eval += 2ull * (k - 1) * found;
                }
            } else if (Q.is_tree) {
                if (k < n)
                    expand_tree(L, list, count, next, &counts[k + 1], w, nw, W.grow, sizeof(W.grow) / 4, ends, lane);
                eval_tree_list<CM>(L, ColexMemo{ranks, L.loff, false}, M, list, count, k, tree_group(count, 64u * nw), 64u * w + lane, 64u * nw);
            } else {
                if (k < n)
                    expand_sets<false>(L, list, count, next, &counts[k + 1], w, nw, expand_group(count, 64u * nw),
                                       W.grow, sizeof(W.grow) / 4, ends, lane);
                // sets per wave at a time, and waves per set, as in the per-level kernel
                const uint32_t per = max(pair_sets(count, nw), min(count, kBatchPer));
                const bool heavy = (1u << k) / 16u >= ((Q.sched >> kSchedHeavyShift) & 0xffffu);
                const uint32_t parts = heavy && 2u * count <= nw ? nw / count : 1u;
                if (walk)
                    eval_subsets<CM>(L, BitMemo{}, M, list, count, k, w, nw, pair_sets(count, nw), parts, W.pairs[wave].p0, pp, lane,
                                     my_ccp, my_eval);
                else
                    eval_pairs<CM, false, false>(L, BitMemo{}, M, list, count, k, w, nw, per, parts, W.pairs[wave], pp, lane, my_ccp,
                               my_eval);
            }
            // the level's memo is complete before the next level reads it
            if (team) failed = !team_barrier(R, size, spread, phase, s_ok);
            else __syncthreads();
            if (t == 0 && member == 0) {
                s_conn += count;
                if (Q.is_tree) {
                    s_ccp += (unsigned long long)(k - 1) * count;
                    s_eval += 2ull * (k - 1) * count;
                }
            }
        }
        // counters of the cyclic queries and unranked tree joins
        for (int off = 32; off >= 1; off >>= 1) {
            my_ccp += (unsigned long long)__shfl_xor((long long)my_ccp, off);
            my_eval += (unsigned long long)__shfl_xor((long long)my_eval, off);
        }
        if (lane == 0 && (my_ccp || my_eval)) {
            atomicAdd(&s_conn, my_sets);  // (found by lane 0 alone)
            atomicAdd(&s_ccp, my_ccp);
            atomicAdd(&s_eval, my_eval);
        }
        __syncthreads();
        if (team) {  // the team's counters meet in its record; the first member finishes the query
            if (t == 0) {
                __hip_atomic_fetch_add(&R->connected, s_conn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_add(&R->ccp, s_ccp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_add(&R->evaluated, s_eval, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (!failed) failed = !team_barrier(R, size, spread, phase, s_ok);
            if (member != 0) continue;
            if (t == 0) {
                s_conn = __hip_atomic_load(&R->connected, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_ccp = __hip_atomic_load(&R->ccp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_eval = __hip_atomic_load(&R->evaluated, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
        }
        double root = 0.0;
        const bool ok = !failed && extract_plan(L.binom, L.loff, !Q.is_tree, M, n, plans + Q.plan_off, &root, W.plan, t, blockDim.x);
        __syncthreads();
        if (t == 0) {
            BatchOut o;
            o.cost = root;
            o.t_start = s_t0;
            o.t_end = (unsigned long long)wall_clock64();
            o.connected = s_conn;
            o.ccp = s_ccp;
            o.evaluated = s_eval;
            o.error = ok ? 0u : 1u;
            o.pad = 0;
            out[Q.out] = o;
        }
        __syncthreads();
    }
}

}  // namespace

hipError_t launch_batch(int cost_model, uint32_t workgroups, const BatchQueryDev *qs,
                        const uint32_t *edges, const double *cards, const double *sels, const double *bcosts,
                        const uint32_t *binom,
                        char *slots, uint64_t slot_bytes, uint32_t maxn, mpdp_plan_node *plans, BatchOut *out,
                        TeamRec *teams, BatchCounters *bc, hipStream_t s) {
    if (cost_model == MPDP_COST_COUT)
        hipLaunchKernelGGL(k_batch<MPDP_COST_COUT>, dim3(workgroups), dim3(kBatchBlock), 0, s, qs, edges, cards,
                           sels, bcosts, binom, slots, slot_bytes, maxn, plans, out, teams, bc);
    else
        hipLaunchKernelGGL(k_batch<MPDP_COST_PGLIKE>, dim3(workgroups), dim3(kBatchBlock), 0, s, qs, edges,
                           cards, sels, bcosts, binom, slots, slot_bytes, maxn, plans, out, teams, bc);
    return hipGetLastError();
}

}  // namespace mpdp
