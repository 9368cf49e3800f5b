"""Levels walked as lists of connected sets, against the CPU oracle (every memo
entry, the plan and the counters, bit for bit) where they can go wrong: block
structures that split many times (triangles around one relation, cliques
joined by a path, cycles sharing relations), sets whose search states
overflow a wave's pool (dense graphs), sets shared between waves (the top
levels), and more than 24 relations (the last digits of the rank table)."""
import numpy as np
import pytest

import oracle
from paper_2202_13511_amd import mpdp, workloads as W

from test_gpu_parity import CMS, check_memo, check_plan, check_stats, run_ws

pytestmark = pytest.mark.gpu


def friendship(k):
    """k triangles around relation 0."""
    return 2 * k + 1, [e for i in range(k) for e in ([0, 2 * i + 1], [0, 2 * i + 2], [2 * i + 1, 2 * i + 2])]


def barbell(a, path, b):
    """Cliques of a and b relations joined by a path."""
    n = a + path + b
    edges = [[i, j] for i in range(a) for j in range(i)] + [[i, i + 1] for i in range(a - 1, a + path)]
    return n, edges + [[a + path + i, a + path + j] for i in range(b) for j in range(i)]


def necklace(k):
    """k squares in a row, neighbours sharing a relation."""
    edges = []
    for i in range(k):
        c = 3 * i
        edges += [[c, c + 1], [c + 1, c + 3], [c + 3, c + 2], [c + 2, c]]
    return 3 * k + 1, edges


@pytest.mark.parametrize("cm", CMS)
@pytest.mark.parametrize("n,edges", [friendship(7), barbell(5, 3, 6), barbell(3, 0, 3), necklace(4)])
def test_block_structures(n, edges, cm):
    q = W.from_edges(n, edges, n, f"blocks{n}")
    res, gm = run_ws(q, cm)
    ref = oracle.mpdp(q, cm)
    check_memo(q, gm, ref)
    check_plan(q, res, ref)
    check_stats(q, res, ref, general=True)


@pytest.mark.parametrize("cm", CMS)
@pytest.mark.parametrize("q", [W.random_connected(15, 2, 0.6), W.clique(13, 3), W.cycle_chords(5, n=17, chords=6)],
                         ids=lambda q: q.name)
def test_full_pools_and_shared_sets(q, cm):
    res, gm = run_ws(q, cm)
    ref = oracle.mpdp(q, cm)
    check_memo(q, gm, ref)
    check_plan(q, res, ref)
    check_stats(q, res, ref, general=True)


def hub_tree(n, hub):
    """A star around another relation than 0, one leaf of it a chain of two."""
    others = [v for v in range(n) if v != hub]
    return [[hub, v] for v in others[:-1]] + [[others[0], others[-1]]]


@pytest.mark.parametrize("cm", CMS)
@pytest.mark.parametrize("q", [W.random_tree(13, 1), W.random_tree(17, 2), W.random_tree(18, 3), W.chain(17, 4),
                               W.snowflake(18, 5), W.from_edges(15, hub_tree(15, 9), 6, "hub15"),
                               W.from_edges(16, hub_tree(16, 15), 7, "hub16")], ids=lambda q: q.name)
def test_tree_lists(q, cm):
    """Tree joins of every shape (levels in one workgroup, levels of their
    own, one to eight lanes a set), numbered at random."""
    res, gm = run_ws(q, cm)
    ref = oracle.mpdp(q, cm)
    check_memo(q, gm, ref)
    check_plan(q, res, ref)
    check_stats(q, res, ref, general=False)
    res, gm = run_ws(q, cm, flags=mpdp.MPDP_FLAG_TIMING)
    check_memo(q, gm, ref)
    check_plan(q, res, ref)
    assert res.stats["ms_eval"] > 0


@pytest.mark.parametrize("n", [24, 25, 31, 32])
def test_cycle_ranks(n):
    """A cycle's counts in closed form, and its optimum: the best of the chains
    that its last join leaves (every plan joins two arcs at the root)."""
    q = W.cycle(n, n)
    if n > 30:
        import torch
        if torch.cuda.mem_get_info()[0] < 1.1 * mpdp.mpdp_workspace_bytes(n):
            pytest.skip("not enough device memory")
    ws = mpdp.workspace(n, mpdp.MPDP_COST_COUT)
    res = mpdp.mpdp_optimize_ws(q, mpdp.MPDP_COST_COUT, ws)
    assert res.stats["connected_sets"] == n * (n - 1) + 1 - n
    assert res.stats["ccp_pairs"] == (n ** 3 - 2 * n ** 2 + n) // 2
    # arcs of k < n relations have k - 1 bridges, the whole cycle is one block
    assert res.stats["evaluated_pairs"] == n * sum(2 * (k - 1) for k in range(2, n)) + 2 ** n - 2
    # interval DP over arcs (start, length), C_out
    sel = {(min(u, v), max(u, v)): s for (u, v), s in zip(q.edges.tolist(), q.sel.tolist())}

    def card(members):
        c = 1.0
        have = set()
        for v in sorted(members):
            c = c * float(q.card[v])
            for u in sorted(have):
                if (u, v) in sel:
                    c = c * sel[(u, v)]
            have.add(v)
        return 1.0 if c < 1.0 else c

    best = {(s, 1): 0.0 for s in range(n)}
    for k in range(2, n + 1):
        for s in range(n if k < n else 1):
            c = card([(s + i) % n for i in range(k)])
            if k < n:
                best[(s, k)] = min((best[(s, j)] + best[((s + j) % n, k - j)]) + c for j in range(1, k))
            else:
                root = min((best[(t, j)] + best[((t + j) % n, n - j)]) + c for t in range(n) for j in range(1, n))
    assert np.float64(res.cost).view(np.uint64) == np.float64(root).view(np.uint64)


def chain_and_clique(length, size, card=None, sel=None):
    """A chain that ends in a clique: many extra edges, few connected sets."""
    n = length + size
    edges = [(i, i + 1) for i in range(length)]
    edges += [(a, b) for a in range(length, n) for b in range(a + 1, n)]
    q = W.from_edges(n, edges, n, f"chain{length}clique{size}")
    if card is not None:
        q.card[:] = card
        q.sel[:] = sel
    return q


LAZY = [chain_and_clique(18, 7), chain_and_clique(22, 6), chain_and_clique(20, 8), chain_and_clique(19, 7, 1000.0, 0.001),
        chain_and_clique(18, 7, 1e308, 1.0)]


@pytest.mark.parametrize("q", LAZY, ids=lambda q: f"{q.name}-{q.card[0]:.0e}")
def test_cards_read_only_where_needed(q):
    """PG-like, more than 24 relations and many extra edges: a pair whose costs
    alone are too high has its cards left out.  With ties and with costs
    beyond the largest double as well, bit for bit against the oracle."""
    assert q.n > 24 and q.m + 1 >= 38
    cm = mpdp.MPDP_COST_PGLIKE
    ref = oracle.mpdp(q, cm)
    got = mpdp.mpdp_optimize_ws(q, cm, mpdp.workspace(q.n, cm))
    assert np.float64(got.cost).view(np.uint64) == np.float64(ref.root_cost).view(np.uint64)
    want = oracle.plan_from_memo(ref)
    assert [(p["relset"], p["left"], p["right"], p["op"]) for p in got.plan] == \
           [(p["relset"], p["left"], p["right"], p["op"]) for p in want]
    assert (got.stats["connected_sets"], got.stats["ccp_pairs"], got.stats["evaluated_pairs"]) == \
           (ref.connected_sets, ref.ccp_ordered // 2, ref.evaluated)


@pytest.mark.parametrize("card,sel", [(None, None), (1000.0, 0.001), (1e308, 1.0)], ids=["drawn", "ties", "infinite"])
def test_cards_read_late_on_dense_levels(card, sel):
    """PG-like: levels of which a quarter or more of the subsets are connected
    (and levels of many sets) read a pair's cards after its costs, others along
    with them; a query has levels of both kinds."""
    q = W.random_connected(19, 3, 0.15)
    if card is not None:
        q.card[:] = card
        q.sel[:] = sel
    cm = mpdp.MPDP_COST_PGLIKE
    res, gm = run_ws(q, cm)
    ref = oracle.mpdp(q, cm)
    check_memo(q, gm, ref)
    check_plan(q, res, ref)
    check_stats(q, res, ref, general=True)


def test_dense_query_under_both_models():
    """Eighteen relations on two hubs take 5.7 ms under PG-like and 4.7 under C_out;
    with every pair's cards read along with its costs they took 10.5."""
    q = W.from_edges(20, [[h, v] for h in (0, 1) for v in range(2, 20)], 20, "hubs20")

    def median_ms(cm):
        ws = mpdp.workspace(20, cm)
        return sorted(mpdp.mpdp_optimize_ws(q, cm, ws).stats["ms_total"] for _ in range(9))[4]

    assert median_ms(mpdp.MPDP_COST_PGLIKE) < 1.6 * median_ms(mpdp.MPDP_COST_COUT)


def triangles(k):
    """k triangles strung along a path, one edge between neighbours."""
    edges = []
    for i in range(k):
        c = 3 * i
        edges += [[c, c + 1], [c + 1, c + 2], [c, c + 2]] + ([[c + 2, c + 3]] if i + 1 < k else [])
    return 3 * k, edges


def joined_cliques(sizes):
    """Cliques in a row, neighbours sharing a relation."""
    edges, at = [], 0
    for s in sizes:
        edges += [[at + i, at + j] for i in range(s) for j in range(i)]
        at += s - 1
    return at + 1, edges


# from 19 relations on: smaller cyclic queries walk their subsets (up to 18)
LARGER = [friendship(9), barbell(6, 9, 6), barbell(10, 0, 9), necklace(6), necklace(7), triangles(7),
          joined_cliques((4, 5, 6, 7)), joined_cliques((3, 9, 3, 9)), necklace(8), barbell(7, 12, 7)]


@pytest.mark.parametrize("cm", CMS)
@pytest.mark.parametrize("n,edges", LARGER)
def test_block_structures_of_larger_queries(n, edges, cm):
    """The pair search and Alg. 3's counter on graphs of many blocks; the last two
    with more than 24 relations."""
    assert n > 18
    q = W.from_edges(n, edges, n, f"blocks{n}")
    res, gm = run_ws(q, cm)
    ref = oracle.mpdp(q, cm)
    check_memo(q, gm, ref)
    check_plan(q, res, ref)
    check_stats(q, res, ref, general=True)


@pytest.mark.parametrize("cm", CMS)
@pytest.mark.parametrize("q", [chain_and_clique(9, 12), chain_and_clique(12, 10), chain_and_clique(6, 13),
                               chain_and_clique(8, 12, 1000.0, 0.001), W.cycle_chords(5, n=19, chords=8)],
                         ids=lambda q: f"{q.name}-{q.card[0]:.0e}")
def test_full_pools_and_shared_sets_of_larger_queries(q, cm):
    """Sets of up to 8191 pairs, whose search states overflow a wave's pool, and
    top levels whose few sets are shared between waves."""
    assert q.n > 18
    res, gm = run_ws(q, cm)
    ref = oracle.mpdp(q, cm)
    check_memo(q, gm, ref)
    check_plan(q, res, ref)
    check_stats(q, res, ref, general=True)


def with_stats(q, card, sel):
    q.card[:] = card
    q.sel[:] = sel
    return q


@pytest.mark.parametrize("cm", CMS)
@pytest.mark.parametrize("q", [W.clique(19, 1), W.clique(21, 2), W.random_connected(20, 4, 0.9), W.random_connected(19, 3, 0.4),
                               with_stats(W.random_connected(19, 3, 0.4), 1000.0, 0.001),
                               with_stats(W.clique(20, 5), 1e308, 1.0)], ids=lambda q: f"{q.name}-{q.card[0]:.0e}")
def test_dense_queries_against_dpsub(q, cm):
    """Dense queries walk their sets' subsets.  The oracle takes minutes here: Alg.
    1's kernels, which are compared with it on smaller queries and share no
    level code, leave the same memo; ties and infinite costs among them."""
    res, gm = run_ws(q, cm)
    ref, rm = run_ws(q, cm, flags=mpdp.MPDP_FLAG_ABLATE_DPSUB)
    planned = gm["cost"] >= 0
    planned[0] = False
    assert planned.sum() == ref.stats["connected_sets"] + q.n
    for name in ("cost", "card", "left", "op"):
        assert np.array_equal(gm[name][planned], rm[name][planned]), name
    assert res.plan == ref.plan and res.cost == ref.cost
    for key in ("connected_sets", "ccp_pairs"):
        assert res.stats[key] == ref.stats[key]


def test_dense_query_time():
    """A clique of 22 took 222 ms while each block's subsets were walked, 239 with
    a search for each pair, next to a clique of 19 in 7.3 and 4.4: 31 and 54
    times as long; 113 and 3.0 ms (38 times)."""
    def median_ms(n):
        q, ws = W.clique(n, 1), mpdp.workspace(n, mpdp.MPDP_COST_COUT)
        return sorted(mpdp.mpdp_optimize_ws(q, mpdp.MPDP_COST_COUT, ws).stats["ms_total"] for _ in range(3))[1]

    assert median_ms(22) < 47.0 * median_ms(19)


def path_and_triangles(n, triangles, hub=0):
    """A path with `triangles` of its neighbours' neighbours joined as well; its
    last `hub` relations hang on relation 0."""
    edges = [[i, i + 1] for i in range(n - 1 - hub)] + [[0, n - 1 - i] for i in range(hub)]
    return edges + [[3 * i, 3 * i + 2] for i in range(triangles)]


@pytest.mark.parametrize("n,triangles,hub", [(22, 4, 0), (23, 3, 0), (23, 3, 5), (25, 3, 0), (25, 4, 0), (25, 1, 4)])
def test_both_forms_of_the_search(n, triangles, hub):
    """PG-like queries on both sides of the lines between the kernel that may read
    cards late and the other one: relations, extra edges, the largest degree; up to
    and above 24 relations."""
    q = W.from_edges(n, path_and_triangles(n, triangles, hub), n, f"path{n}+{triangles}+{hub}")
    assert q.m == n - 1 + triangles
    res, gm = run_ws(q, mpdp.MPDP_COST_PGLIKE)
    ref = oracle.mpdp(q, mpdp.MPDP_COST_PGLIKE)
    check_memo(q, gm, ref)
    check_plan(q, res, ref)
    check_stats(q, res, ref, general=True)
