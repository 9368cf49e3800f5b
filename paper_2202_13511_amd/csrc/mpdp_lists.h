// Levels as lists of connected sets: the next level's list is grown from
// this one's (expand_sets), and a set's csg-cmp pairs are enumerated
// directly (eval_pairs: one search step per pair, whatever the block
// structure of the set), instead of unranking every k-subset and testing
// every subset of every block; where most subsets are connected, by a walk
// over the set's subsets (eval_subsets).  Shared by the per-level kernels and
// the batched kernel.  Internal; every function is inlined into its kernels.
#pragma once

#include "mpdp_device.h"

namespace mpdp {
namespace {

// ---------------------------------------------------------------- colex ranks by table

// Colex rank of a set from its six-bit digits: digit j holds relations
// 6j .. 6j + 5 and contributes sum C(6j + b, c + i + 1) over its set bits b
// (i-th from below), where c members of the set lie below the digit.  That
// depends on (j, c, digit) alone: 4284 words for all 32 relations, six
// lookups a set (four up to 24 relations) with no loop over the members.
// (Eight-bit digits would take four lookups but 53 KB of LDS.)
constexpr int kRankAt[6] = {0, 64, 512, 1344, 2560, 4160};
constexpr int kRankWords = 4160 + 31 * 4;
constexpr int kRankWords24 = 2560;  // the first four digits: up to 24 relations

struct RankTable {
    uint32_t v[kRankWords];
};

constexpr RankTable make_rank_table() {
    uint32_t binom[33][34] = {};
    for (int a = 0; a <= 32; ++a) {
        binom[a][0] = 1;
        for (int b = 1; b <= a; ++b) binom[a][b] = binom[a - 1][b - 1] + (b <= a - 1 ? binom[a - 1][b] : 0u);
    }
    RankTable t{};
    for (int j = 0; j < 6; ++j) {
        const int bits = j < 5 ? 6 : 2;
        for (int c = 0; c <= 6 * j; ++c)
            for (int d = 0; d < (1 << bits); ++d) {
                uint32_t r = 0;
                int i = c;
                for (int b = 0; b < bits; ++b)
                    if ((d >> b) & 1) {
                        ++i;
                        r += binom[6 * j + b][i];
                    }
                t.v[kRankAt[j] + (c << bits) + d] = r;
            }
    }
    return t;
}

__device__ const RankTable kRankTable = make_rank_table();

// Copy the digits that n relations need into LDS.
__device__ __forceinline__ void stage_ranks(uint32_t *dst, uint32_t n) {
    const uint32_t words = n <= 24 ? kRankWords24 : kRankWords;
    const uint4 *src = reinterpret_cast<const uint4 *>(kRankTable.v);
    for (uint32_t i = threadIdx.x; i < words / 4; i += blockDim.x) reinterpret_cast<uint4 *>(dst)[i] = src[i];
}
static_assert(kRankWords % 4 == 0 && kRankWords24 % 4 == 0, "the rank table is copied in 16-byte units");

__device__ __forceinline__ uint32_t colex_rank(const uint32_t *T, uint32_t X, bool wide) {
    uint32_t r = T[X & 63u];
    r += T[64 + (popc32(X & 0x3fu) << 6) + ((X >> 6) & 63u)];
    r += T[512 + (popc32(X & 0xfffu) << 6) + ((X >> 12) & 63u)];
    r += T[1344 + (popc32(X & 0x3ffffu) << 6) + ((X >> 18) & 63u)];
    if (wide) {  // uniform: more than 24 relations
        r += T[2560 + (popc32(X & 0xffffffu) << 6) + ((X >> 24) & 63u)];
        r += T[4160 + (popc32(X & 0x3fffffffu) << 2) + (X >> 30)];
    }
    return r;
}

// nbrs of a set of up to 24 relations: three lookups.
template <bool kWide>
__device__ __forceinline__ uint32_t nbrs_of(const uint32_t (*nb)[256], uint32_t V) {
    const uint32_t r = nb[0][V & 255u] | nb[1][(V >> 8) & 255u] | nb[2][(V >> 16) & 255u];
    return kWide ? r | nb[3][V >> 24] : r;
}

// Where a set's memo entry is.  ColexMemo: the level's offset plus the colex
// rank, the layout that callers see.  BitMemo: the set itself, for a memo of
// the kernel's own, with no lookup at all.
struct ColexMemo {
    const uint32_t *T;
    const uint64_t *loff;
    bool wide;  // more than 24 relations (T holds the last digits only then)
    __device__ __forceinline__ uint64_t operator()(uint32_t X, uint32_t k) const {
        return loff[k] + colex_rank(T, X, wide);
    }
};
struct BitMemo {
    __device__ __forceinline__ uint64_t operator()(uint32_t X, uint32_t) const { return X; }
};

// ---------------------------------------------------------------- buffers

// One wave's LDS.  The pool is the stack of search states (eval_pairs):
// kPoolN entries are shared by all lanes, kReserve more are for the one lane
// that goes on alone when the pool is full.  With 28 relations and 10 chords
// the sets have hundreds of pairs, which fill 512 entries now and then; at
// 192 some waves spent most of their time stalled (8.0 -> 12.3 ms).  The batched
// kernel's queries are smaller, and two of its workgroups share a CU's LDS.
template <uint32_t kPoolN, uint32_t kReserve>
struct PairBufN {
    static constexpr uint32_t kPool = kPoolN;
    uint32_t p0[kPoolN + kReserve], p1[kPoolN + kReserve], p2[kPoolN + kReserve];
    unsigned long long bc[64];  // best key of each set: cost bits,
    double card[64];            // card(S)
    uint32_t bl[64], bop[64];   // left set, operator
    uint32_t claim[64];
    uint8_t slot[kPoolN + kReserve];
};
using PairBuf = PairBufN<448, 64>;

// ---------------------------------------------------------------- Alg. 3's counter

// Sum over the blocks of G[S] (S connected) of 2^b - 2, Alg. 3's
// EvaluatedCounter: relations of degree one are bridges (2 each) and are
// stripped; in what remains every cut vertex that a block hangs on has three
// or more neighbours, so only those are tested, by whether their neighbours
// reach each other without them; a cut splits the rest in two pieces that
// share the vertex.  A relation that is no cut of a piece is none of the
// pieces that come of it, so each is tested once, and the one cut at again in
// the piece that may hold more of its components.  One lane per set; `todo` holds the pieces put aside (16 per lane, stride 64; a
// piece put aside has two or more relations that the others lack, so 32
// relations leave at most 15).  (28 relations, 10 chords: 21 % of the level
// kernels' time with a test of every relation of every piece.)
template <bool kWide>
__device__ __forceinline__ unsigned long long block_candidates(const LdsGraph &L, uint32_t S, uint32_t *todo) {
    unsigned long long sum = 0;
    uint32_t sp = 0, K = S, untested = S;
    // relations of degree one from v on: v, its neighbour if that leaves it
    // with one edge, ..
    const auto strip = [&](uint32_t &P, uint32_t v) {
        while (P & v) {
            const uint32_t nv = L.adj[ctz32(v)] & P;
            if (nv == 0 || (nv & (nv - 1))) break;
            sum += 2;
            P ^= v;
            v = nv;
        }
    };
    for (uint32_t U = K; U; U &= U - 1) strip(K, lowbit(U));
    for (;;) {
        uint32_t cur = 0, nv = 0;
        for (uint32_t U = untested & K; U != 0u; U &= U - 1u) {
            cur = lowbit(U);
            nv = L.adj[ctz32(cur)] & K;
            if (popc32(nv) >= 3) break;
            untested ^= cur;
            cur = 0;
        }
        if (cur == 0u) {
            if (K & (K - 1)) sum += (1ull << popc32(K)) - 2ull;
            if (sp == 0) return sum;
            --sp;
            K = todo[sp * 64];
            continue;
        }
        const uint32_t b = 31u - (uint32_t)__builtin_clz(nv), C = K ^ cur;
        uint32_t fa = L.adj[ctz32(nv)] & C, fb = L.adj[b] & C, sa = lowbit(nv) | fa, sb = (1u << b) | fb;
        while ((sa & sb) == 0u && fa != 0u && fb != 0u) {
            fa = nbrs_of<kWide>(L.nb, fa) & C & ~sa;
            fb = nbrs_of<kWide>(L.nb, fb) & C & ~sb;
            sa |= fa;
            sb |= fb;
        }
        const bool met = (sa & sb) != 0u;
        uint32_t seen = met ? sa | sb : fa == 0u ? sa : sb, fr = met ? fa | fb : 0u;
        while (fr != 0u && (nv & ~seen) != 0u) {
            fr = nbrs_of<kWide>(L.nb, fr) & C & ~seen;
            seen |= fr;
        }
        if ((nv & ~seen) == 0u) {
            untested ^= cur;
            continue;
        }
        uint32_t piece = seen | cur;  // seen: a component without cur
        K &= ~seen;
        strip(piece, cur);
        strip(K, cur);
        if (piece & (piece - 1)) {
            todo[sp * 64] = piece;
            ++sp;
        }
    }
}

// ---------------------------------------------------------------- csg-cmp pairs of any connected set

// All csg-cmp pairs of the sets list[0 .. count), Alg. 3's result without
// its candidate subsets.  For one set S with lowest relation r, a search
// state (A, X), A holding r, stands for every pair whose left side contains
// A and none of X; S - A is connected, so (A, S - A) itself is one of them.
// The others take some neighbour of A into the left side, and are divided by
// the first one they take: for v the lowest neighbour of A in S - A - X,
// v joins A, or v joins X and the next neighbour is tried.  When v joins A,
// the component of S - A - v that holds X (or, while X is empty, each
// component in turn) becomes the right side and everything else the left,
// which is again connected; if v separates X there is no such pair.  So
// every state but those dead ends yields one pair: 1.2 to 1.5 steps per
// pair on cycles with chords (n = 24), 1.0 on cliques, where the walk over
// all subsets of a block tests up to 632 candidates per pair.
//
// A wave takes `per` sets at a time; their states share one LDS stack, from
// which idle lanes pop and onto which a lane pushes the state it leaves
// behind.  A full stack stalls the lanes that would push, all but the first
// active one, which goes on depth first into the reserve (a search path
// pushes less than two states per relation, so 64 entries suffice) until
// there is room.  The memo reads of a pair are issued one step before they
// are used (with kLazy, PG-like, its costs first, its cards if still needed), and a lane keeps the best key of the set it is on to itself
// until it comes to another set.
//
// With parts > 1 (levels of few sets) `parts` waves share one set: each runs
// the same first steps until there are at least two states per part, keeps
// every parts-th state, and leaves its key in `rec`; the last one to arrive
// reduces them.
//
// A lane's state: A, C = S - A, X and F, the neighbours of A in C - X still
// to try.  F = 0 with C != 0 marks components still to place: the right
// sides are the components of C, and A = S - C.  C = 0: idle.  When v joins
// A, the relations that become its neighbours are those of v alone (the
// components that go left with it touch nothing of the one that stays).
// A stack entry is three bit planes (A: 1 0 0, C alone: 0 1 0, X: 1 1 0,
// F: 0 0 1) and the set's slot.
struct PairState {
    uint32_t A, C, X, F, slot;
};

template <class Buf>
__device__ __forceinline__ void push_state(Buf &B, uint32_t at, uint32_t A, uint32_t C, uint32_t X, uint32_t F,
                                           uint32_t slot) {
    B.p0[at] = A | X;
    B.p1[at] = C & ~F;
    B.p2[at] = F;
    B.slot[at] = (uint8_t)slot;
}

template <int CM>
struct PairLoad {
    double cA, cB, kA, kB;
    uint64_t ia, ib;  // entries of A and B
    uint32_t A, B, slot;
    bool on;
};

// A lane's best key of the set in `slot`, not yet in the set's LDS entry.
struct PairBest {
    unsigned long long c;
    uint32_t l, op, slot;
    double card;
};

__device__ __forceinline__ bool key_before(unsigned long long c, uint32_t l, uint32_t op, unsigned long long bc,
                                           uint32_t bl, uint32_t bop) {
    return (c < bc) | ((c == bc) & ((l < bl) | ((l == bl) & (op < bop))));
}

// The keys of the lanes in `on` into their sets' entries (LDS, this wave's
// alone); lanes that improve the same set take turns.
template <class Buf>
__device__ __forceinline__ void flush_best(Buf &B, const PairBest &b, bool on, uint32_t lane) {
    bool better = on && key_before(b.c, b.l, b.op, B.bc[b.slot], B.bl[b.slot], B.bop[b.slot]);
    while (__ballot(better) != 0ull) {
        if (better) B.claim[b.slot] = lane;
        wave_sync_lds();
        if (better && B.claim[b.slot] == lane) {
            B.bc[b.slot] = b.c;
            B.bl[b.slot] = b.l;
            B.bop[b.slot] = b.op;
            better = false;
        }
        wave_sync_lds();
        better = better && key_before(b.c, b.l, b.op, B.bc[b.slot], B.bl[b.slot], B.bop[b.slot]);
    }
}

// The pair whose memo values have arrived into its lane's best key.
template <int CM, class Buf>
__device__ __forceinline__ void settle_pair(Buf &B, const PairLoad<CM> &p, PairBest &b, uint32_t lane) {
    const bool moved = p.on && p.slot != b.slot;
    if (__ballot(moved) != 0ull) {
        flush_best(B, b, moved, lane);
        if (moved) {
            b.c = ~0ull;
            b.l = b.op = ~0u;
            b.slot = p.slot;
            b.card = B.card[p.slot];
        }
    }
    if (!p.on) return;
    unsigned long long c;
    uint32_t l, op;
    const double base = p.cA + p.cB, cS = b.card;
    if (CM == MPDP_COST_COUT) {
        c = (unsigned long long)__double_as_longlong(base + cS);
        l = p.A < p.B ? p.A : p.B;
        op = MPDP_OP_JOIN;
    } else {
        const double out = 0.01 * cS;
        const double hjA = ((base + 0.0125 * p.kB) + 0.0025 * p.kA) + out;  // A outer, B hashed
        const double nlA = (base + (0.0025 * p.kA) * p.kB) + out;
        const double hjB = ((base + 0.0125 * p.kA) + 0.0025 * p.kB) + out;  // B outer, A hashed
        const double nlB = (base + (0.0025 * p.kB) * p.kA) + out;
        const bool hA = hjA <= nlA, hB = hjB <= nlB;
        const unsigned long long ca = (unsigned long long)__double_as_longlong(hA ? hjA : nlA);
        const unsigned long long cb = (unsigned long long)__double_as_longlong(hB ? hjB : nlB);
        const bool first = (ca < cb) | ((ca == cb) & (p.A < p.B));
        c = first ? ca : cb;
        l = first ? p.A : p.B;
        op = (first ? hA : hB) ? MPDP_OP_HASH : MPDP_OP_NESTLOOP;
    }
    if (key_before(c, l, op, b.c, b.l, b.op)) {
        b.c = c;
        b.l = l;
        b.op = op;
    }
}

// kLazy, PG-like: a pair whose costs have arrived in `p` goes on to `q`, which reads
// its cards, unless its cost alone is too high: every offer adds terms of
// zero or more to cA + cB, then card(S)'s, and rounding keeps the order, so
// (cA + cB) + 0.01 card(S) bounds them all from below.  Most pairs end here,
// which leaves out half of their gathers, for a step more of latency.
template <int CM, class Buf>
__device__ __forceinline__ void pass_pair(const Buf &B, const MemoPtrs &M, const PairLoad<CM> &p, PairLoad<CM> &q,
                                          const PairBest &b) {
    q.on = p.on;
    if (!p.on) return;
    const unsigned long long least =
        (unsigned long long)__double_as_longlong((p.cA + p.cB) + 0.01 * B.card[p.slot]);
    unsigned long long bound = B.bc[p.slot];
    if (p.slot == b.slot && b.c < bound) bound = b.c;
    q.on = least <= bound;
    if (!q.on) return;
    q.cA = p.cA;
    q.cB = p.cB;
    q.A = p.A;
    q.B = p.B;
    q.slot = p.slot;
    q.kA = M.card[p.ia];
    q.kB = M.card[p.ib];
}

struct PairParts {
    HeavyPart *rec;     // (global memory, or LDS where one workgroup's waves share)
    uint32_t *arrived;  // per set, zero between uses
};

template <int CM, bool kWide, bool kLazy, class At, class Buf>
__device__ void eval_pairs(const LdsGraph &L, const At &at_of, const MemoPtrs &M, const uint32_t *list,
                           uint32_t count, uint32_t k, uint32_t w, uint32_t nw, uint32_t per, uint32_t parts,
                           Buf &B, PairParts pp, uint32_t lane, unsigned long long &ccp,
                           unsigned long long &evaluated) {
    const unsigned long long below = (1ull << lane) - 1ull;
    const uint32_t chunks = (count + per - 1) / per, items = parts > 1 ? count * parts : chunks;
    for (uint32_t item = w; item < items; item += nw) {
        // sets s0, s0 + chunks, ..: neighbours in the list have much the same
        // number of pairs, and no wave should get the largest ones alone
        const uint32_t s0 = parts > 1 ? item / parts : item, part = parts > 1 ? item - s0 * parts : 0u;
        const uint32_t ns = parts > 1 ? 1u : (count - s0 + chunks - 1u) / chunks;
        bool quiet = part != 0;       // the first steps of a shared set count for its first part alone
        bool shared = parts > 1;      // not split yet
        uint32_t myset = 0;
        double mycard = 0.0;
        PairBest best{~0ull, ~0u, ~0u, lane, 0.0};
        if (lane < ns) {
            myset = list[s0 + lane * chunks];
            if (part == 0) evaluated += block_candidates<kWide>(L, myset, B.p0 + lane);
            tree_card_n<1>(L, &myset, k, &mycard);
            B.card[lane] = mycard;
            B.bc[lane] = ~0ull;
            B.bl[lane] = B.bop[lane] = ~0u;
        }
        // the first right sides are the components of S without its lowest
        // relation: every lane starts with its set
        PairState s{lowbit(myset), myset & (myset - 1u), 0u, 0u, lane};
        best.card = mycard;
        if (shared) best.card = rdlane_f64(mycard, 0);
        uint32_t top = 0;
        PairLoad<CM> ld;
        ld.on = false;
        ld.slot = 0;
        ld.A = ld.B = 0;
        ld.cA = ld.cB = ld.kA = ld.kB = 0.0;
        ld.ia = ld.ib = 0;
        PairLoad<CM> ld2 = ld;  // (kLazy) the pair whose cards are on the way
        wave_sync_lds();
        for (;;) {
            if (top != 0u) {  // idle lanes take states from the stack
                const unsigned long long im = __ballot(s.C == 0u);
                const uint32_t r = (uint32_t)__popcll(im & below);
                if (s.C == 0u && r < top) {
                    const uint32_t e = top - 1u - r;
                    const uint32_t e0 = B.p0[e], e1 = B.p1[e], e2 = B.p2[e];
                    s.slot = B.slot[e];
                    s.A = e0 & ~e1;
                    s.X = e0 & e1;
                    s.C = e1 | e2;
                    s.F = e2;
                }
                const uint32_t ni = (uint32_t)__popcll(im);
                top = top > ni ? top - ni : 0u;
            }
            const unsigned long long am = __ballot(s.C != 0u);
            if (am == 0ull) break;
            if (shared && top + (uint32_t)__popcll(am) >= 2u * parts) {
                // every parts-th state is this part's
                shared = quiet = false;
                if (lane % parts != part) s.C = 0u;
                const uint32_t keep = top > part ? (top - part + parts - 1u) / parts : 0u;
                for (uint32_t i0 = 0; i0 < keep; i0 += 64u) {
                    const uint32_t i = i0 + lane;
                    const uint32_t from = part + i * parts;
                    uint32_t e0 = 0, e1 = 0, e2 = 0;
                    if (i < keep) { e0 = B.p0[from]; e1 = B.p1[from]; e2 = B.p2[from]; }
                    wave_sync_lds();
                    if (i < keep) { B.p0[i] = e0; B.p1[i] = e1; B.p2[i] = e2; B.slot[i] = 0; }
                    wave_sync_lds();
                }
                top = keep;
                continue;
            }
            // one step of every active lane
            const bool act = s.C != 0u, place = s.F == 0u;  // place: the next component of C
            const uint32_t v = lowbit(s.F), rest = s.F ^ v, C1 = s.C ^ v;
            const uint32_t av = L.adj[ctz32(v | 0x80000000u)];
            const uint32_t nv = place ? C1 : av & C1;
            uint32_t comp = C1;
            if ((nv & (nv - 1u)) != 0u) {
                // C was connected, so C1 is once one neighbour of v reaches the
                // others, and every component of C1 holds one.  Two neighbours
                // search towards each other: they meet in half as many rounds
                // as one would need, and apart, the smaller component ends it.
                const uint32_t b = 31u - (uint32_t)__builtin_clz(nv);
                uint32_t sa = lowbit(nv), sb = 1u << b;
                uint32_t fa = L.adj[ctz32(sa)] & C1, fb = L.adj[b] & C1;
                sa |= fa;
                sb |= fb;
                while ((sa & sb) == 0u && fa != 0u && fb != 0u) {
                    fa = nbrs_of<kWide>(L.nb, fa) & C1 & ~sa;
                    fb = nbrs_of<kWide>(L.nb, fb) & C1 & ~sb;
                    sa |= fa;
                    sb |= fb;
                }
                const bool met = (sa & sb) != 0u;
                // met: one component, which may lack others; apart: that of
                // the side that ended
                uint32_t seen = met ? sa | sb : fa == 0u ? sa : sb;
                uint32_t fr = met ? fa | fb : 0u;
                while (fr != 0u && (nv & ~seen) != 0u) {
                    fr = nbrs_of<kWide>(L.nb, fr) & C1 & ~seen;
                    seen |= fr;
                }
                if ((nv & ~seen) != 0u) {
                    if (s.X != 0u && (s.X & seen) == 0u) {  // the component of X is the one that stays
                        const uint32_t others = nv & ~seen;
                        if ((others & (others - 1u)) == 0u) {
                            seen = C1 & ~seen;
                        } else {
                            seen = lowbit(s.X);
                            fr = seen;
                            while (fr != 0u) {
                                fr = nbrs_of<kWide>(L.nb, fr) & C1 & ~seen;
                                seen |= fr;
                            }
                        }
                    }
                    comp = seen;
                }
            }
            const bool ok = act && C1 != 0u && (s.X & ~comp) == 0u;
            const uint32_t left = s.X == 0u ? C1 & ~comp : 0u;  // other components, each a right side of its own
            const bool push_rest = ok && rest != 0u, push_left = ok && left != 0u;
            const unsigned long long mr = __ballot(push_rest), ml = __ballot(push_left);
            uint32_t at = top + (uint32_t)__popcll(mr & below) + (uint32_t)__popcll(ml & below);
            uint32_t total = (uint32_t)__popcll(mr) + (uint32_t)__popcll(ml);
            bool go = act;
            if (top + total > Buf::kPool) {  // uniform, rare
                const uint32_t need = (push_rest ? 1u : 0u) + (push_left ? 1u : 0u);
                go = act && (need == 0u || at + need <= Buf::kPool || (am & below) == 0ull);
                total = (uint32_t)__popcll(__ballot(go && push_rest)) + (uint32_t)__popcll(__ballot(go && push_left));
            }
            top += total;
            if (!kLazy) {
                settle_pair<CM>(B, ld, best, lane);
            } else {
                settle_pair<CM>(B, ld2, best, lane);
                pass_pair<CM>(B, M, ld, ld2, best);
            }
            ld.on = go && ok && !quiet;
            if (go && ok) {
                const uint32_t S = s.A | s.C, A1 = S & ~comp;
                if (push_rest) push_state(B, at++, s.A, s.C, s.X | v, rest, s.slot);
                if (push_left) push_state(B, at, S & ~left, left, 0u, 0u, s.slot);
                if (!quiet) {
                    const uint32_t ka = (uint32_t)popc32(A1);
                    const uint64_t ia = at_of(A1, ka);
                    const uint64_t ib = at_of(comp, k - ka);
                    ld.A = A1;
                    ld.B = comp;
                    ld.slot = s.slot;
                    ld.cA = M.cost[ia];
                    ld.cB = M.cost[ib];
                    if (kLazy) {
                        ld.ia = ia;
                        ld.ib = ib;
                    } else if (CM != MPDP_COST_COUT) {
                        ld.kA = M.card[ia];
                        ld.kB = M.card[ib];
                    }
                    ++ccp;
                }
                s.F = ((place ? nbrs_of<kWide>(L.nb, s.A) : av) | rest) & comp & ~s.X;
                s.A = A1;
                s.C = s.F != 0u ? comp : 0u;
            } else if (go) {  // no pair takes v to the left
                s.X |= v;
                s.F = rest;
                s.C = rest != 0u ? s.C : 0u;
            }
            wave_sync_lds();
        }
        if (kLazy) {
            settle_pair<CM>(B, ld2, best, lane);
            pass_pair<CM>(B, M, ld, ld2, best);
            ld = ld2;
        }
        settle_pair<CM>(B, ld, best, lane);
        flush_best(B, best, true, lane);
        wave_sync_lds();
        if (parts == 1) {
            if (lane < ns) {
                const uint64_t at = at_of(myset, k);
                store_best(M, at, Key{B.bc[lane], B.bl[lane], B.bop[lane]}, mycard);
            }
        } else {
            // the part's key, then the last part to arrive takes the least
            // (a part of which no state was left keeps the worst key)
            const uint32_t S0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)myset);
            HeavyPart *rec = pp.rec + (size_t)s0 * parts;
            uint32_t n_here = 0;
            if (lane == 0) {
                unsigned long long *r64 = reinterpret_cast<unsigned long long *>(&rec[part]);
                __hip_atomic_store(&r64[0], B.bc[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&r64[1], ((unsigned long long)B.bop[0] << 32) | B.bl[0], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
                // the record is all that others read, and its stores are
                // device-wide themselves: once they are complete, the
                // arrival may follow (an agent-scope release would write
                // the whole L2 back first, in every part's wave)
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_s_waitcnt(0);
                n_here = __hip_atomic_fetch_add(&pp.arrived[s0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            n_here = (uint32_t)__builtin_amdgcn_readfirstlane((int)n_here);
            if (n_here == parts - 1u) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");  // (device-wide loads follow)
                Key best = worst_key();
                for (uint32_t p = lane; p < parts; p += 64u) {
                    unsigned long long *r64 = reinterpret_cast<unsigned long long *>(&rec[p]);
                    const unsigned long long c =
                        __hip_atomic_load(&r64[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const unsigned long long lo =
                        __hip_atomic_load(&r64[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const Key o{c, (uint32_t)lo, (uint32_t)(lo >> 32)};
                    if (key_less(o, best)) best = o;
                }
                best = wave_min(best);
                if (lane == 0) {
                    store_best(M, at_of(S0, k), best, mycard);
                    __hip_atomic_store(&pp.arrived[s0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        wave_sync_lds();
    }
}

// ---------------------------------------------------------------- the next level's sets

// The waves of a workgroup collect the sets that they find in LDS (`buf`, `cap`
// words, 64 or more) and append them with one atomic on the list's end: some 30
// ns each when all workgroups add to one word, an atomic per 64 sets or per wave
// made that word the bound of the smaller levels.
struct ExpandEnds {
    uint32_t fill, end, start;  // words taken, first word not used, place in the list
    uint32_t more;              // (expand_tree) a wave waits for room
};

// The connected sets of k + 1 relations from the `count` of k relations in
// `list`: S + v for every neighbour v of S.  Such a set arises once per
// relation whose removal leaves it connected; it is kept where v is the
// highest relation of the last round of a breadth-first search from its
// lowest relation (which can always be removed), so that every set is listed
// once.  One search per neighbour, against C(n, k + 1) subsets to unrank and
// search; `group` lanes (a power of two) divide the neighbours of one set.
// Sets that the workgroup's buffer has no room for go straight to the list,
// an atomic per step.  Starts and ends with the workgroup in step.
template <bool kWide>
__device__ void expand_sets(const LdsGraph &L, const uint32_t *list, uint32_t count, uint32_t *out, uint32_t *out_count,
                            uint32_t w, uint32_t nw, uint32_t group, uint32_t *buf, uint32_t cap, ExpandEnds &ends,
                            uint32_t lane) {
    const unsigned long long below = (1ull << lane) - 1ull;
    const uint32_t each = 64u / group, sub = lane & (group - 1u);
    if (threadIdx.x == 0) ends = ExpandEnds{0u, cap, 0u, 0u};
    __syncthreads();
    for (uint32_t base = w * each; base < count; base += nw * each) {
        const uint32_t i = base + lane / group;
        const uint32_t S = i < count ? list[i] : 0u;
        uint32_t N = nbrs_of<kWide>(L.nb, S) & ~S;
        for (uint32_t j = 0; j < sub; ++j) N &= N - 1u;
        while (__ballot(N != 0u) != 0ull) {
            const uint32_t v = lowbit(N), S1 = S | v;
            for (uint32_t j = 0; j < group; ++j) N &= N - 1u;
            bool keep = false;
            if (v != 0u) {
                uint32_t seen = lowbit(S1), fr = seen;
                while (seen != S1) {  // S1 is connected
                    fr = nbrs_of<kWide>(L.nb, fr) & S1 & ~seen;
                    seen |= fr;
                }
                keep = (v & fr) != 0u && (fr & ~(v | (v - 1u))) == 0u;
            }
            const unsigned long long m = __ballot(keep);
            const uint32_t add = (uint32_t)__popcll(m);
            if (add == 0u) continue;
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&ends.fill, add);
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
            if (at + add <= cap) {
                if (keep) buf[at + (uint32_t)__popcll(m & below)] = S1;
            } else {  // the buffer is full: straight to the list
                if (lane == 0) {
                    atomicMin(&ends.end, at);
                    at = atomicAdd(out_count, add);
                }
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
                if (keep) out[at + (uint32_t)__popcll(m & below)] = S1;
            }
        }
    }
    __syncthreads();
    const uint32_t have = min(ends.fill, ends.end);
    if (threadIdx.x == 0 && have != 0u) ends.start = atomicAdd(out_count, have);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < have; i += blockDim.x) out[ends.start + i] = buf[i];
    __syncthreads();
}

// The same for a tree join's sets in preorder numbers, for which the sets that
// add a child numbered above every member are all there is to list (a set's
// last relation in preorder has no child in it), without any search.  A wave
// that finds the buffer full keeps its place and goes on once the workgroup has
// emptied it: finding sets is so quick here that their atomics bound the level
// (straight to the list, a star of 25 around relation 12 took 8.7 ms).
__device__ __forceinline__ void expand_tree(const LdsGraph &L, const uint32_t *list, uint32_t count, uint32_t *out,
                                            uint32_t *out_count, uint32_t w, uint32_t nw, uint32_t *buf, uint32_t cap,
                                            ExpandEnds &ends, uint32_t lane) {
    const unsigned long long below = (1ull << lane) - 1ull;
    uint32_t base = w * 64u, S = 0, N = 0;  // the wave's next sets; this lane's set and its children still to add
    if (threadIdx.x == 0) ends = ExpandEnds{0u, cap, 0u, 0u};
    __syncthreads();
    for (;;) {
        for (;;) {
            const unsigned long long m = __ballot(N != 0u);
            if (m == 0ull) {
                if (base >= count) break;
                S = base + lane < count ? list[base + lane] : 0u;
                N = nbrs(L.pch, S) & ~(0xffffffffu >> __builtin_clz(S | 1u));
                base += nw * 64u;
                continue;
            }
            const uint32_t add = (uint32_t)__popcll(m);
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&ends.fill, add);
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
            if (at + add > cap) {  // full; so is it for whoever comes next
                if (lane == 0) {
                    atomicMin(&ends.end, at);
                    ends.more = 1u;
                }
                break;
            }
            if (N) buf[at + (uint32_t)__popcll(m & below)] = S | lowbit(N);
            N &= N - 1u;
        }
        __syncthreads();
        const uint32_t have = min(ends.fill, ends.end), more = ends.more;
        if (threadIdx.x == 0 && have != 0u) ends.start = atomicAdd(out_count, have);
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < have; i += blockDim.x) out[ends.start + i] = buf[i];
        __syncthreads();
        if (more == 0u) return;
        if (threadIdx.x == 0) ends = ExpandEnds{0u, cap, 0u, 0u};
        __syncthreads();
    }
}

// ---------------------------------------------------------------- best keys of lane groups

// A set's best key so far: the smallest cost (+inf before the first offer;
// every connected set has a finite one or offers +inf itself), then the
// smallest left set, which names the offer and its operator (a set's offers
// all have different left sets).
struct SetBest {
    double c;
    uint32_t l, op;
};

__device__ __forceinline__ void take_best(SetBest &b, const SetBest &o) {
    const bool take = (o.c < b.c) | ((o.c == b.c) & (o.l < b.l));
    b.c = take ? o.c : b.c;
    b.l = take ? o.l : b.l;
    b.op = take ? o.op : b.op;
}

template <int kCtrl>
__device__ __forceinline__ void merge_best(SetBest &b) {
    const unsigned long long c = (unsigned long long)__double_as_longlong(b.c);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)c, kCtrl, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(c >> 32), kCtrl, 0xf, 0xf, true);
    SetBest o;
    o.c = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    o.l = (uint32_t)__builtin_amdgcn_mov_dpp((int)b.l, kCtrl, 0xf, 0xf, true);
    o.op = (uint32_t)__builtin_amdgcn_mov_dpp((int)b.op, kCtrl, 0xf, 0xf, true);
    take_best(b, o);
}

// The best of 2^lgP neighbouring lanes, in all of them.
__device__ __forceinline__ void group_best(SetBest &b, uint32_t P) {
    if (P >= 2u) merge_best<0xB1>(b);   // lanes ^ 1 (quad_perm 1 0 3 2)
    if (P >= 4u) merge_best<0x4E>(b);   // ^ 2 (quad_perm 2 3 0 1)
    if (P >= 8u) merge_best<0x141>(b);  // ^ 4: quads agree, so mirroring eight lanes swaps them
    if (P >= 16u) merge_best<0x140>(b); // ^ 8, mirroring a row
    for (uint32_t d = 16; d < P; d <<= 1) {
        SetBest o;
        o.c = __shfl_xor(b.c, (int)d, 64);
        o.l = (uint32_t)__shfl_xor((int)b.l, (int)d, 64);
        o.op = (uint32_t)__shfl_xor((int)b.op, (int)d, 64);
        take_best(b, o);
    }
}

// Both offers of the pair (A, B) under PG-like, or its one under C_out.
template <int CM>
__device__ __forceinline__ SetBest pair_best(uint32_t A, uint32_t B, double cA, double cB, double kA, double kB,
                                             double cS) {
    const double base = cA + cB;
    SetBest o;
    if (CM == MPDP_COST_COUT) {
        o.c = base + cS;
        o.l = A < B ? A : B;
        o.op = MPDP_OP_JOIN;
    } else {
        const double out = 0.01 * cS;
        const double hjA = ((base + 0.0125 * kB) + 0.0025 * kA) + out;  // A outer, B hashed
        const double nlA = (base + (0.0025 * kA) * kB) + out;
        const double hjB = ((base + 0.0125 * kA) + 0.0025 * kB) + out;  // B outer, A hashed
        const double nlB = (base + (0.0025 * kB) * kA) + out;
        const bool hA = hjA <= nlA, hB = hjB <= nlB;
        o.c = hA ? hjA : nlA;
        o.l = A;
        o.op = hA ? MPDP_OP_HASH : MPDP_OP_NESTLOOP;
        const SetBest o2{hB ? hjB : nlB, B, hB ? MPDP_OP_HASH : MPDP_OP_NESTLOOP};
        take_best(o, o2);
    }
    return o;
}

// The keys of one set's `parts` parts meet in pp.rec: true, with the best of all
// in `best`, in lane 0 of the part that comes last.
__device__ __forceinline__ bool meet_parts(const PairParts &pp, uint32_t set, uint32_t part, uint32_t parts, SetBest &best,
                                           uint32_t lane) {
    HeavyPart *rec = pp.rec + (size_t)set * parts;
    uint32_t n_here = 0;
    if (lane == 0) {
        unsigned long long *r64 = reinterpret_cast<unsigned long long *>(&rec[part]);
        __hip_atomic_store(&r64[0], (unsigned long long)__double_as_longlong(best.c), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&r64[1], ((unsigned long long)best.op << 32) | best.l, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        // (device-wide stores, complete before the arrival)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        n_here = __hip_atomic_fetch_add(&pp.arrived[set], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    n_here = (uint32_t)__builtin_amdgcn_readfirstlane((int)n_here);
    if (n_here != parts - 1u) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    SetBest o{__builtin_inf(), ~0u, ~0u};
    if (lane < parts) {
        unsigned long long *r64 = reinterpret_cast<unsigned long long *>(&rec[lane]);
        const unsigned long long c = __hip_atomic_load(&r64[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned long long l = __hip_atomic_load(&r64[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        o = SetBest{__longlong_as_double((long long)c), (uint32_t)l, (uint32_t)(l >> 32)};
    }
    group_best(o, 64u);
    best = o;
    if (lane == 0) __hip_atomic_store(&pp.arrived[set], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return lane == 0;
}

// ---------------------------------------------------------------- subsets of sets, dense graphs

// The csg-cmp pairs of the sets list[0 .. count) where most subsets are
// connected: every subset that holds the set's lowest relation, A = lowest +
// x, and the rest of the set.  The memo holds a cost below zero where there is
// no plan, so that the two gathers that a pair's cost takes are its test as
// well; neighbouring lanes take neighbouring subsets.  Up to six relations
// 2^(k-1) lanes take a set, from seven on a wave does, or `parts` waves.
// PG-like reads the cards of pairs whose costs leave them a chance (see
// pass_pair).  Bound by the gathers; the search (eval_pairs) takes a chain of
// dependent steps for each pair, here the next subset waits for nothing.
template <int CM, class At>
__device__ void eval_subsets(const LdsGraph &L, const At &at_of, const MemoPtrs &M, const uint32_t *list, uint32_t count, uint32_t k,
                             uint32_t w, uint32_t nw, uint32_t per, uint32_t parts, uint32_t *todo, PairParts pp,
                             uint32_t lane, unsigned long long &ccp, unsigned long long &evaluated) {
    // subsets of a lane in flight (PG-like, four cost the batched kernel
    // registers that all its paths then miss, 5 to 10 %)
    constexpr int kEach = CM == MPDP_COST_COUT ? 4 : 2;
    const uint32_t chunks = (count + per - 1u) / per, items = parts > 1u ? count * parts : chunks;
    const uint32_t lgP = k < 7u ? k - 1u : 6u, P = 1u << lgP, sub = lane & (P - 1u), sets = 64u >> lgP;
    const uint32_t all = k < 7u ? 1u : 1u << (k - 7u);  // rounds of P subsets
    for (uint32_t item = w; item < items; item += nw) {
        const uint32_t s0 = parts > 1u ? item / parts : item, part = parts > 1u ? item - s0 * parts : 0u;
        const uint32_t ns = parts > 1u ? 1u : (count - s0 + chunks - 1u) / chunks;
        const uint32_t rounds = part < all ? (all - part + parts - 1u) / parts : 0u;
        uint32_t myset = 0;
        double mycard = 0.0;
        if (lane < ns) {
            myset = list[s0 + lane * chunks];
            if (part == 0u) evaluated += block_candidates<false>(L, myset, todo + lane);
            tree_card_n<1>(L, &myset, k, &mycard);
        }
        for (uint32_t j = 0; j < ns; j += sets) {
            const int from = (int)(j + (lane >> lgP));
            const uint32_t S = (uint32_t)__shfl((int)myset, from, 64), lo = lowbit(S), rest = S ^ lo;
            const double cS = __shfl(mycard, from, 64);
            const uint32_t step = all > parts ? deposit(64u * parts, rest) : 0u;
            uint32_t x = deposit(part * 64u + sub, rest);
            SetBest best{__builtin_inf(), ~0u, ~0u};
            for (uint32_t r = 0; r < rounds; r += kEach) {
                uint32_t A[kEach];
                uint64_t ia[kEach], ib[kEach];
                double cA[kEach], cB[kEach];
#pragma unroll
                for (int u = 0; u < kEach; ++u) {
                    const bool in = r + (uint32_t)u < rounds && x != rest;
                    A[u] = in ? lo | x : 0u;  // (the empty set has no plan)
                    x = ((x | ~rest) + step) & rest;  // (the masked add carries through the holes)
                    const uint32_t ka = (uint32_t)popc32(A[u]);
                    ia[u] = in ? at_of(A[u], ka) : 0ull;
                    ib[u] = in ? at_of(S ^ A[u], k - ka) : 0ull;
                    cA[u] = M.cost[ia[u]];
                    cB[u] = M.cost[ib[u]];
                }
#pragma unroll
                for (int u = 0; u < kEach; ++u) {
                    const bool on = cA[u] >= 0.0 && cB[u] >= 0.0;
                    ccp += on ? 1u : 0u;
                    const uint32_t B = S ^ A[u];
                    if (CM == MPDP_COST_COUT) {
                        SetBest o = pair_best<CM>(A[u], B, cA[u], cB[u], 0.0, 0.0, cS);
                        o.l = on ? o.l : ~0u;
                        o.c = on ? o.c : __builtin_inf();
                        take_best(best, o);
                    } else if (on && (cA[u] + cB[u]) + 0.01 * cS <= best.c) {
                        take_best(best, pair_best<CM>(A[u], B, cA[u], cB[u], M.card[ia[u]], M.card[ib[u]], cS));
                    }
                }
            }
            group_best(best, P);
            bool store = S != 0u && sub == 0u;
            if (parts > 1u) store = meet_parts(pp, s0, part, parts, best, lane);
            if (store)
                store_best(M, at_of(S, k), Key{(unsigned long long)__double_as_longlong(best.c), best.l, best.op}, cS);
        }
    }
}

// ---------------------------------------------------------------- tree joins

// Alg. 2 for the sets list[0 .. count) of a tree join (in preorder numbers),
// 2^lgP lanes a set:
// with the tree rooted at relation 0, the edge (parent(c), c) of G[S] gives
// the pair (S and c's subtree, the rest) for every member c whose parent is
// a member.  The lanes of a group take every 2^lgP-th member, four at a time
// with all their reads in flight; a member without a pair (the topmost, or
// past the end) reads entry 0 and offers nothing.  `thread` of `threads`
// (groups of lanes never straddle waves).
template <int CM, class At>
__device__ void eval_tree_list(const LdsGraph &L, const At &at_of, const MemoPtrs &M,
                               const uint32_t *list, uint32_t count, uint32_t k, uint32_t lgP, uint32_t thread,
                               uint32_t threads) {
    const uint32_t P = 1u << lgP, sub = thread & (P - 1u);
    for (uint32_t i = thread >> lgP; i < count; i += threads >> lgP) {
        const uint32_t S = nbrs(L.perm, list[i]);
        double cS;
        tree_card_n<1>(L, &S, k, &cS);
        double bc = __builtin_inf();
        uint32_t bl = ~0u, bop = ~0u, U = S;
        for (uint32_t j = 0; j < sub; ++j) U &= U - 1u;
        while (U) {
            uint32_t A[4];
            uint64_t ia[4], ib[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t c = (uint32_t)ctz32(U | 0x80000000u);
                const uint2 pd = *reinterpret_cast<const uint2 *>(L.pd[c]);  // parent bit, subtree
                A[u] = U != 0u && (S & pd.x) != 0u ? pd.y & S : 0u;
                for (uint32_t j = 0; j < P; ++j) U &= U - 1u;
                const uint32_t ka = (uint32_t)popc32(A[u]);
                ia[u] = A[u] ? at_of(A[u], ka) : 0ull;
                ib[u] = A[u] ? at_of(S ^ A[u], k - ka) : 0ull;
            }
            double cA[4], cB[4], kA[4], kB[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                cA[u] = M.cost[ia[u]];
                cB[u] = M.cost[ib[u]];
                kA[u] = CM == MPDP_COST_COUT ? 0.0 : M.card[ia[u]];
                kB[u] = CM == MPDP_COST_COUT ? 0.0 : M.card[ib[u]];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t B = S ^ A[u];
                const double base = cA[u] + cB[u];
                double c;
                uint32_t l, op;
                if (CM == MPDP_COST_COUT) {
                    c = base + cS;
                    l = A[u] < B ? A[u] : B;
                    op = MPDP_OP_JOIN;
                } else {
                    const double out = 0.01 * cS;
                    const double hjA = ((base + 0.0125 * kB[u]) + 0.0025 * kA[u]) + out;  // A outer, B hashed
                    const double nlA = (base + (0.0025 * kA[u]) * kB[u]) + out;
                    const double hjB = ((base + 0.0125 * kA[u]) + 0.0025 * kB[u]) + out;  // B outer, A hashed
                    const double nlB = (base + (0.0025 * kB[u]) * kA[u]) + out;
                    const bool hA = hjA <= nlA, hB = hjB <= nlB;
                    const double ca = hA ? hjA : nlA, cb = hB ? hjB : nlB;
                    const bool first = (ca < cb) | ((ca == cb) & (A[u] < B));
                    c = first ? ca : cb;
                    l = first ? A[u] : B;
                    op = (first ? hA : hB) ? MPDP_OP_HASH : MPDP_OP_NESTLOOP;
                }
                // a set's offers all have different left sets, so cost and
                // left set order them
                const bool take = A[u] != 0u && ((c < bc) | ((c == bc) & (l < bl)));
                bc = take ? c : bc;
                bl = take ? l : bl;
                bop = take ? op : bop;
            }
        }
        for (uint32_t d = 1; d < P; d <<= 1) {
            const double oc = __shfl_xor(bc, (int)d, 64);
            const uint32_t ol = (uint32_t)__shfl_xor((int)bl, (int)d, 64), oo = (uint32_t)__shfl_xor((int)bop, (int)d, 64);
            const bool take = (oc < bc) | ((oc == bc) & (ol < bl));
            bc = take ? oc : bc;
            bl = take ? ol : bl;
            bop = take ? oo : bop;
        }
        if (sub == 0u)
            store_best(M, at_of(S, k),
                       Key{(unsigned long long)__double_as_longlong(bc), bl, bop}, cS);
    }
}

// Relation u's share of the list of two-relation sets of a tree join: in
// preorder numbers, u and each of its children.  A relation's edge to its
// parent sits at the relation's number less one.
__device__ __forceinline__ void first_tree_list(const LdsGraph &L, uint32_t u, uint32_t *list2) {
    for (uint32_t C = nbrs(L.pch, 1u << u); C; C &= C - 1u) list2[ctz32(C) - 1] = (1u << u) | lowbit(C);
}

// Lanes per set (2^0 .. 2^3): as many as `threads` lanes leave the level.
__device__ __forceinline__ uint32_t tree_group(uint32_t count, uint32_t threads) {
    uint32_t lgP = 0;
    while (lgP < 3u && (2u * count << lgP) <= threads) ++lgP;
    return lgP;
}

// Sets that a wave of eval_pairs takes at a time, of a level of `count` sets
// and nw waves: the same for all waves, so that none goes another round for
// the last few sets.  (A step's latency bounds a level, not its lanes: half
// as many waves with twice the sets took cycles with chords 10 % longer.)
__device__ __forceinline__ uint32_t pair_sets(uint32_t count, uint32_t nw) {
    const uint32_t rounds = (count + 64u * nw - 1u) / (64u * nw);
    return (count + rounds * nw - 1u) / (rounds * nw);
}

// Lanes that grow one set's successors (expand_sets).
__device__ __forceinline__ uint32_t expand_group(uint32_t count, uint32_t threads) {
    uint32_t group = 1;
    while (group < 16u && 2u * count * group <= threads) group <<= 1;
    return group;
}

}  // namespace
}  // namespace mpdp
