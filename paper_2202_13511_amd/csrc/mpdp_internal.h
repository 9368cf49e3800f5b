// Internal interface between the host runtime (mpdp_host.cpp) and the gfx950
// kernels (mpdp_kernels.hip).  Not part of the public C-ABI.
#pragma once

#include <cstddef>
#include <cstdint>

#include <hip/hip_runtime.h>

#include "mpdp.h"

namespace mpdp {

constexpr int kMaxRel = 32;

// Per-workgroup copy of the query information, laid out on the host exactly
// as the kernels keep it in LDS so that staging is a plain 16-byte copy.
// The kernels that work on lists of connected sets read only the prefix
// before the preorder tables (kListLdsBytes).
struct LdsImage {
    uint64_t loff[34];                        // memo offset of level k: sum of C(n, j), j < k
    double card[kMaxRel];
    double bcost[kMaxRel];                    // cost of scanning relation v under the model
    double csel[kMaxRel][2];                  // per v: card[v], then sel(lowest u < v adjacent to v, v) (1.0 without one)
    uint32_t lo[kMaxRel][2];                  // per v: bit of its lowest neighbour u < v (0 without one), its other neighbours u < v
    uint32_t adj[kMaxRel];                    // bit u of adj[v]: edge (u, v)
    uint32_t pd[kMaxRel][2];                  // tree joins rooted at 0, per v: bit of its parent (0 at the root),
                                              // then the relations of the subtree rooted at v
    uint32_t selrow[kMaxRel];                 // first sel entry of relation v
    double sel[kMaxRel * (kMaxRel - 1) / 2];  // per v: sel(u, v) of edges u < v, u ascending
    uint32_t nb[4][256];                      // neighbours of a set, one table per bitmap byte
    uint32_t pch[4][256];                     // tree joins, relations numbered in preorder from relation 0: children of
                                              // a set, per byte
    uint32_t perm[4][256];                    // and the set in the query's own numbers, per byte
    uint32_t ch[4][256];                      // tree joins rooted at 0: children of a set, per byte
    uint32_t binom[33 * 33];                  // C(a, b) at [a * 33 + b]
    uint32_t pad[3];
};
static_assert(offsetof(LdsImage, csel) % 16 == 0, "(card, sel) pairs are read as 16-byte units");
static_assert(offsetof(LdsImage, lo) % 8 == 0, "lowest-neighbour pairs are read as 8-byte units");
static_assert(offsetof(LdsImage, pd) % 8 == 0, "(parent, subtree) pairs are read as 8-byte units");
static_assert(offsetof(LdsImage, sel) % 16 == 0, "the image is copied in parts of 16-byte units");
static_assert(offsetof(LdsImage, pch) % 16 == 0 && offsetof(LdsImage, ch) % 16 == 0,
              "the image is copied in parts of 16-byte units");
constexpr size_t kListLdsBytes = offsetof(LdsImage, pch);
static_assert(sizeof(LdsImage) % 16 == 0, "LdsImage is copied in 16-byte units");

// Query information as the kernels read it.  Built on the host, uploaded
// once per call.
struct DevGraph {
    LdsImage lds;
    uint32_t n, m, is_tree, cost_model;
    uint32_t ablate;                     // kAblateDpsub: every connected set is one block (DPSUB's enumeration)
    uint32_t flat;                       // tree joins whose tree, rooted at relation 0, has depth one
    uint32_t pad[2];
};

// Memo, level-compact: the entry of a relation set S sits at
// level_off[|S|] + colex(S), colex(S) = sum over the i-th smallest member s_i
// of S (i from 0) of C(s_i, i + 1).  One contiguous slab per level.
struct MemoPtrs {
    double *cost;
    double *card;
    uint32_t *left;
    uint8_t *op;
};

// Device-side counters, cleared by the init kernel.
struct Counters {
    uint32_t level_count[34];   // connected sets found at each level (DPSUB ablation: none)
    uint32_t general_count[34]; // DPSUB ablation: connected sets of each level
    uint32_t heavy_count[34];   // sets handed to the heavy kernel at each level
    uint32_t prune_slots[34];   // unfused-prune ablation: sets whose pair keys were written at each level
    uint32_t extract_error;     // nonzero if plan extraction met an inconsistent memo
    uint32_t pad;
    unsigned long long evaluated; // Alg. 3 candidates (general path)
    unsigned long long ccp;       // unordered csg-cmp pairs (general path)
};

// Small queries (mpdp_small.hip): one launch for the whole query.  The query
// travels in the kernel's arguments; sel(u, v), u < v, at v (v - 1) / 2 + u,
// 1.0 without an edge.  out: pinned host memory, or device
// memory that is copied back.  memo.cost null: the memo is not kept.
constexpr uint32_t kSmallMaxRel = 12;  // 2^12 entries of 23 bytes fit in LDS, 2^13 do not

struct SmallQuery {
    uint32_t n, is_tree;
    uint32_t adj[kSmallMaxRel], kids[kSmallMaxRel];  // kids: a tree join's children, rooted at 0
    uint32_t pd[kSmallMaxRel][2];
    uint32_t loff[16];
    double card[kSmallMaxRel], bcost[kSmallMaxRel];
    double sel[kSmallMaxRel * (kSmallMaxRel - 1) / 2];
};

struct SmallOut {
    unsigned long long connected, ccp, evaluated;
    double root;
    uint32_t error, pad;
    mpdp_plan_node plan[2 * kSmallMaxRel - 1];
};

hipError_t launch_small(const SmallQuery &q, int cost_model, MemoPtrs memo, SmallOut *out, hipStream_t s);

// Where a query's results go: pinned host memory, or the device region they
// are copied back from.
struct Results {
    Counters *cnt;
    mpdp_plan_node *plan;
    double *root;
};

// Batched path (mpdp_batch.hip): one queue entry per workgroup at a time.
// A query is one entry, or, if it is large, up to kTeamSize entries in a row:
// a team of workgroups that share its levels.
struct BatchQueryDev {
    uint32_t n, m, is_tree, cost_model;
    uint64_t card_off, edge_off, plan_off;
    uint32_t sched, out;       // the query's schedule (packed as below); index of its BatchOut
    uint32_t team, pad0;       // entries, and so most workgroups, of the query (1: no team)
    uint32_t team_rec, pad;    // the team's TeamRec (team > 1)
};

// Shared state of one team, zero at the start of a launch.  The first
// workgroup that joins leads: it publishes its memo slot, which the whole team
// uses, and closes the team when all have joined or some time has passed; the
// level's list counts live here instead of in LDS.
struct TeamRec {
    uint32_t joined;                 // workgroups that have joined; kTeamClosed once no more may
    uint32_t formed;                 // set by the leader: the team's workgroups, kTeamSpread if on several XCDs
    uint32_t arrive;                 // barrier arrivals so far
    uint32_t slot;                   // workgroup whose slot holds the memo and lists
    uint32_t error;                  // a barrier wait ran out of time
    uint32_t xcds;                   // bit x: a member runs on XCD x
    uint32_t count[24];              // connected sets per level k
    unsigned long long connected, ccp, evaluated;
};
constexpr uint32_t kTeamClosed = 1u << 31, kTeamSpread = 1u << 31;

constexpr uint32_t kTeamSize = 8;     // largest team
constexpr uint32_t kTeamMinRel = 17;  // only queries of at least this many relations may get a team

// Schedule of one query in the batched kernel: bits 0-1 hold log2 of the
// consecutive ranks per lane of a star's levels (1, 2 or 4), bits 8-23 the
// number of 16-subset chunks from which a cyclic query's sets may be shared
// by several waves.  Bits 2 and 3, set by the host from the query's shape: a
// tree join's levels are unranked (kSchedUnrank), a cyclic query's sets are
// walked subset by subset (kSchedWalk).
constexpr uint32_t kSchedChunkMask = 3u;
constexpr uint32_t kSchedUnrank = 4u, kSchedWalk = 8u;
constexpr uint32_t kSchedHeavyShift = 8;
constexpr uint32_t kSchedDefault = 2u | (256u << kSchedHeavyShift);

struct BatchOut {
    double cost;
    unsigned long long t_start, t_end;  // device wall clock at the query's start and end
    unsigned long long connected, ccp, evaluated;
    uint32_t error, pad;
};

// The queue: the teams in a share for each XCD, entries share_end[x - 1] ..
// share_end[x] - 1 (from 0 for the first), then the others for all.  The
// workgroups of an XCD start with its share, so that a team's members,
// neighbours there, run on one XCD.  What the workgroups count in lies on
// lines of its own: accesses to one line take turns, some 30 ns each.
struct BatchCounters {
    uint32_t entries;        // queue entries of this launch
    uint32_t share_end[8];
    alignas(128) uint32_t next;            // next entry to take after the shares
    alignas(128) unsigned long long t0;    // earliest workgroup start (device wall clock)
    alignas(128) uint32_t share_taken[8];
};

constexpr uint32_t kBatchMaxRel = 20;      // largest query the batched path takes
static_assert(kBatchMaxRel < 24, "TeamRec holds the counts of levels up to 23");
constexpr uint32_t kBatchWorkgroups = 512; // persistent workgroups (two per CU)

hipError_t launch_batch(int cost_model, uint32_t workgroups, const BatchQueryDev *qs,
                        const uint32_t *edges, const double *cards, const double *sels, const double *bcosts,
                        const uint32_t *binom, char *slots, uint64_t slot_bytes, uint32_t maxn,
                        mpdp_plan_node *plans, BatchOut *out, TeamRec *teams,
                        BatchCounters *bc, hipStream_t s);

// Waves of a level that walks lists of connected sets, which is also the
// most parts its sets are shared out in (HeavyPart records and arrival
// counters, zeroed by launch_init and left at zero by every level).  tally:
// csg-cmp pairs and Alg. 3 candidates per workgroup, zeroed by launch_init,
// summed by launch_extract (null there: not used).  list2:
// where the connected sets of two relations go (null: no lists; `preorder`:
// those of a tree join, in preorder numbers).
constexpr uint32_t kPairGrid = 256;            // one workgroup per CU
constexpr uint32_t kPairBlock = 1024;
constexpr uint32_t kPairWaves = kPairGrid * (kPairBlock / 64);

// src: the query in pinned host memory, brought to g on the way (null: g holds
// it already).
hipError_t launch_init(const DevGraph *src, DevGraph *g, uint32_t n, MemoPtrs memo, uint32_t *list2,
                       uint32_t *arrived, unsigned long long *tally, bool preorder, Counters *cnt, hipStream_t s);
struct HeavyPart;
// Cyclic queries of up to kBitsMaxRel relations: launch_bits_init (after
// launch_init) fills conn, list, card and the single relations' cost; one
// launch_bits_level a level.  sets: C(n, k), the most the level can have.
// At 18 relations, C_out, a clique takes 1074 us here and 1742 with lists and
// pair search, a cycle with 4 chords 331 and 530; each relation more triples
// the candidates.  At 19 (limit 19 against 18) this path still takes 330 us
// for a bare cycle against 414, but 1080 against 628 with 8 chords, 1870
// against 525 for a star with one edge more, and 3869 for a clique against
// the subset walk's 2841.
constexpr uint32_t kBitsMaxRel = 18;
struct BitsSpace {
    uint32_t *conn;       // bit S: S is connected
    double *cost, *card;  // of a connected set S, at S * stride: two arrays, or (PG-like) pairs
    uint32_t stride;
    uint32_t *cand;       // its Alg. 3 candidates (sum over its blocks of 2^b - 2)
    uint32_t *list;       // connected sets, level k from loff[k] on
};
hipError_t launch_bits_init(const DevGraph *g, uint32_t n, Counters *cnt, const BitsSpace &b, hipStream_t s);
hipError_t launch_bits_level(const DevGraph *g, int cost_model, uint32_t n, uint32_t k, uint64_t sets,
                             const Counters *cnt, const BitsSpace &b, MemoPtrs memo, HeavyPart *rec, uint32_t *arrived,
                             unsigned long long *tally, hipStream_t s);

// One level of a tree join, or levels k0 .. k1 by one workgroup (with k0 = 2
// in place of launch_init).  even, odd: the lists of even and odd levels, in
// preorder numbers; count: the sets of level k.
constexpr uint32_t kTreeListGrid = 1024;
hipError_t launch_tree_level(const DevGraph *g, int cost_model, uint32_t n, uint32_t k, uint64_t count,
                             const uint32_t *list, uint32_t *next, Counters *cnt, MemoPtrs memo, hipStream_t s);
hipError_t launch_tree_span(const DevGraph *src, DevGraph *g, int cost_model, bool star, uint32_t n, uint32_t k0,
                            uint32_t k1, uint32_t *even, uint32_t *odd, Counters *cnt, MemoPtrs memo, hipStream_t s);
// Nearly two edges a relation: only such graphs have many connected subsets
// that make pairs.
inline bool many_edges(uint32_t n, uint32_t m) { return m + 4 >= 2 * n; }
// One level of a cyclic query: the sets of k relations in `list`
// (cnt->level_count[k] of them) evaluated, the sets of k + 1 into `next`.
// lazy (PG-like): levels of many sets read cards late, see lazy_level.
bool lazy_query(uint32_t n, uint32_t m, const uint32_t *adj);
hipError_t launch_level_pairs(const DevGraph *g, int cost_model, bool lazy, uint32_t n, uint32_t k,
                              const uint32_t *list, uint32_t *next, Counters *cnt, MemoPtrs memo, HeavyPart *rec,
                              uint32_t *arrived, unsigned long long *tally, hipStream_t s);
// The same for dense queries of up to kWalkMaxRel relations, subset by subset,
// after launch_no_plans (before launch_init).
constexpr uint32_t kWalkMaxRel = 24;
hipError_t launch_no_plans(MemoPtrs memo, uint32_t n, hipStream_t s);
hipError_t launch_level_walk(const DevGraph *g, int cost_model, uint32_t n, uint32_t k, const uint32_t *list,
                             uint32_t *next, Counters *cnt, MemoPtrs memo, HeavyPart *rec, uint32_t *arrived,
                             unsigned long long *tally, hipStream_t s);
hipError_t launch_filter(const DevGraph *g, uint32_t k, uint64_t ncand, uint32_t *list, Counters *cnt,
                         hipStream_t s);
constexpr uint32_t kAblateDpsub = 1u;

hipError_t launch_level_tree(const DevGraph *g, int cost_model, uint32_t n, uint32_t k, uint64_t ncand, bool compact,
                             bool flat, Counters *cnt, MemoPtrs memo, hipStream_t s);

// Unfused-prune ablation of a tree level (measurement only): the evaluate
// kernel writes the key of every pair of every connected set (16 bytes,
// k per set, slot-major) and the set's record, a separate prune kernel
// reduces each set's keys and writes its memo entry.  pair_keys holds at
// least C(n, k) * k keys, set_recs C(n, k) records.
struct PruneRec {
    uint32_t rank, set;
    double card;
};
struct PairKey {
    unsigned long long c;
    uint32_t l, op;
};
hipError_t launch_level_tree_unfused(const DevGraph *g, int cost_model, uint32_t k, uint64_t ncand, bool flat,
                                     Counters *cnt, MemoPtrs memo, PairKey *pair_keys, PruneRec *set_recs,
                                     hipStream_t s);
// Key and card of one part of a heavy set split over several workgroups.
struct HeavyPart {
    unsigned long long c;
    uint32_t l, op;
    double card;
    double pad;
};
constexpr uint32_t kHeavyGrid = 768;  // workgroups of the heavy-set kernel (three per CU)

// Workgroups per heavy set: one while a level has at least one heavy set
// per workgroup, else as many as share the grid evenly.
__host__ __device__ inline uint32_t heavy_parts(uint32_t count, uint32_t grid) {
    return (count == 0 || count >= grid) ? 1u : grid / count;
}

hipError_t launch_eval_general(const DevGraph *g, int cost_model, uint32_t k, uint64_t ncand,
                               const uint32_t *list, uint32_t *heavy, Counters *cnt, MemoPtrs memo, HeavyPart *parts,
                               hipStream_t s);
hipError_t launch_extract(const DevGraph *g, uint32_t n, MemoPtrs memo, Results down,
                          const unsigned long long *tally, Counters *cnt, hipStream_t s);

}  // namespace mpdp
