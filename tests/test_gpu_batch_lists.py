"""Batched queries level by level: lists of connected sets, stars without
lists, sets shared by waves, teams of workgroups on tree joins as well.  Costs
and plans bit for bit against single-query calls (themselves checked against
the oracle), and the summed counters."""
import numpy as np
import pytest

from paper_2202_13511_amd import mpdp
from paper_2202_13511_amd import workloads as W

pytestmark = pytest.mark.gpu


def hub_last(n, seed):
    """A star whose hub is not relation 0."""
    q = W.star(n, seed)
    edges = [(n - 1 - u, n - 1 - v) for u, v in q.edges.tolist()]
    return W.from_edges(n, [tuple(sorted(e)) for e in edges], seed, f"hub{n}")


def shapes(room):
    trees = [W.star(n, n) for n in (2, 3, 8, 13, 16, 17, 19, 20)] + [hub_last(n, n) for n in (2, 9, 17, 18)]
    trees += [W.chain(n, n) for n in (1, 2, 5, 17, 20)] + [W.snowflake(n, n) for n in (8, 17, 19)]
    trees += [W.random_tree(n, n) for n in (6, 15, 18, 20)]
    dense = [W.clique(n, n) for n in (3, 4, 8, 12, 13)] + [W.cycle_chords(n, n=n, chords=c) for n, c in ((12, 6), (16, 9))]
    large = [W.cycle_chords(40 + i, n=17 + i % 4, chords=i % 3) for i in range(room)]
    return trees + dense + large


@pytest.mark.parametrize("room", [0, 9])  # cyclic queries of 17 or more relations: room for teams
@pytest.mark.parametrize("cm", [mpdp.MPDP_COST_COUT, mpdp.MPDP_COST_PGLIKE])
def test_batched_levels_match_single_calls(cm, room):
    queries = shapes(room)
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


@pytest.mark.parametrize("schedule", [(1, 1), (2, 64), (4, 65535)])
def test_batched_schedules_agree(schedule):
    queries = shapes(3)
    ws = mpdp.batch_workspace(queries)
    base = mpdp.mpdp_optimize_batch(queries, mpdp.MPDP_COST_PGLIKE, ws)
    res = mpdp.mpdp_optimize_batch(queries, mpdp.MPDP_COST_PGLIKE, ws, schedules=[schedule] * len(queries))
    assert np.array_equal(res.costs, base.costs) and res.plans == base.plans
