"""The batched kernel where a batch is made of one kind of query: tiny ones,
tree joins of many connected sets, which are unranked instead of listed, and
dense cyclic ones, whose sets are walked subset by subset."""
import statistics

import pytest

from paper_2202_13511_amd import mpdp, workloads as W

pytestmark = pytest.mark.gpu

COUT, PG = mpdp.MPDP_COST_COUT, mpdp.MPDP_COST_PGLIKE


def kernel_ms(queries, cm):
    """Median device time of a batch's launch."""
    ws = mpdp.batch_workspace(queries)
    run = lambda: mpdp.mpdp_optimize_batch(queries, cm, ws, flags=mpdp.MPDP_FLAG_TIMING).stats["ms_kernel"]
    run()
    return statistics.median(run() for _ in range(9))


@pytest.mark.parametrize("cm", [COUT, PG])
def test_tiny_queries_one_per_workgroup(cm):
    """A workgroup's start, its look for an entry and its end are all that 500
    queries of one relation take.  They took 6.3 times as long as 16 (107 and
    17 us) while every workgroup looked at eight shares that were empty, next to
    the counter that all of them add to; then 2.0 times (27 and 14 us)."""
    assert kernel_ms([W.chain(1, i) for i in range(500)], cm) < 4.0 * kernel_ms([W.chain(1, i) for i in range(16)], cm)


def star_around(n, hub, seed=0):
    return W.from_edges(n, [(min(hub, v), max(hub, v)) for v in range(n) if v != hub], seed, f"star{n}at{hub}")


def two_stars(a, b):
    edges = [(0, 1)] + [(0, 2 + i) for i in range(a)] + [(1, 2 + a + i) for i in range(b)]
    return W.from_edges(a + b + 2, edges, a, f"stars{a}and{b}")


def check_against_single_calls(queries, cm):
    ws = mpdp.batch_workspace(queries)
    res = mpdp.mpdp_optimize_batch(queries, cm, ws)
    conn = ccp = evaluated = 0
    for q, cost, plan in zip(queries, res.costs, res.plans):
        one = mpdp.mpdp_optimize(q, cm)
        assert cost == one.cost and plan == one.plan, q.name
        conn += one.stats["connected_sets"]
        ccp += one.stats["ccp_pairs"]
        evaluated += one.stats["evaluated_pairs"]
    assert (res.stats["connected_sets"], res.stats["ccp_pairs"], res.stats["evaluated_pairs"]) == (conn, ccp, evaluated)


@pytest.mark.parametrize("cm", [COUT, PG])
@pytest.mark.parametrize("room", [0, 6])  # cyclic queries of 17 or more relations: room for teams of trees, too
def test_trees_of_many_sets(room, cm):
    queries = [star_around(n, h, n) for n, h in ((14, 13), (15, 1), (16, 7), (17, 16), (18, 4), (20, 19))]
    queries += [two_stars(a, b) for a, b in ((6, 7), (7, 7), (4, 12), (9, 9))]
    queries += [W.cycle_chords(50 + i, n=17 + i % 3, chords=1) for i in range(room)]
    big = star_around(17, 3, 1)
    big.card[:] = 1e300  # two relations exceed the largest double: every plan ties
    big.sel[:] = 1.0
    check_against_single_calls(queries + [big], cm)


@pytest.mark.parametrize("cm", [COUT, PG])
def test_trees_of_many_sets_time(cm):
    """600 stars of 18 around relation 9 take less than two and a half times as long
    as around relation 0 (3.6 to 4.0 ms and 2.2, PG-like 4.9 to 5.3 and 3.5); as
    lists they took 7.7 and 11.5."""
    assert kernel_ms([star_around(18, 9, i) for i in range(600)], cm) < \
        2.5 * kernel_ms([star_around(18, 0, i) for i in range(600)], cm)


def two_hubs(k):
    """k relations joined to both of relations 0 and 1."""
    return W.from_edges(k + 2, [(h, 2 + i) for h in (0, 1) for i in range(k)], k, f"hubs{k}")


@pytest.mark.parametrize("cm", [COUT, PG])
@pytest.mark.parametrize("room", [0, 1])  # (one: a clique of 17, or all the large ones in teams)
def test_dense_queries(room, cm):
    queries = [W.clique(15, 1), W.clique(16, 2), W.random_connected(15, 3, 0.5), W.random_connected(16, 4, 0.8),
               two_hubs(13), two_hubs(14), W.all_equal_clique(15)]
    if room:
        queries += [W.clique(17, 5), W.random_connected(17, 6, 0.6), W.random_connected(18, 7, 0.3), W.cycle_chords(8, n=18, chords=2)]
    huge = W.clique(15, 9)
    huge.card[:] = 1e300  # costs beyond the largest double: every plan ties
    huge.sel[:] = 1.0
    part = W.random_connected(15, 10, 0.6)
    part.card[::3] = 1e308  # some of them
    check_against_single_calls(queries + [huge, part], cm)


@pytest.mark.parametrize("cm", [COUT, PG])
def test_dense_queries_time(cm):
    """A clique of 16 in a batch, on one workgroup: 17 ms for eight of them,
    PG-like 29 (141 and 160 with a search for each pair), next to 0.29 and 0.31
    ms as a single call on the whole chip."""
    q = W.clique(16, 1)
    ws = mpdp.workspace(16, cm)
    one = statistics.median(mpdp.mpdp_optimize_ws(q, cm, ws).stats["ms_total"] for _ in range(9))
    assert kernel_ms([W.clique(16, i) for i in range(8)], cm) < 200.0 * one


@pytest.mark.parametrize("flags", [0x200, 0x400, 0x600])  # (internal: largest teams, three workgroups, both)
@pytest.mark.parametrize("cm", [COUT, PG])
def test_teams_with_room_for_few_workgroups(cm, flags):
    """A team goes on with the workgroups that have come after a while: with
    three in all, the members that eight entries wait for never come (the launch
    used to end in MPDP_EDEVICE after two seconds), and the entries that are
    taken later are dropped."""
    queries = [W.cycle_chords(70 + i, n=17 + i % 3, chords=i % 4) for i in range(9)] + [W.random_connected(17, 3, 0.4)]
    queries += [star_around(17, 5, 1), W.star(18, 2), W.random_tree(18, 3), W.chain(6, 4), W.clique(9, 5)]
    ws = mpdp.batch_workspace(queries)
    want = mpdp.mpdp_optimize_batch(queries, cm, ws)
    got = mpdp.mpdp_optimize_batch(queries, cm, ws, flags=flags)
    assert got.costs == want.costs and got.plans == want.plans
    for key in ("connected_sets", "ccp_pairs", "evaluated_pairs"):
        assert got.stats[key] == want.stats[key]
