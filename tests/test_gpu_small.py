"""Queries that run as one launch of one workgroup, against the CPU oracle
(every memo entry, plan and counters, bit for bit) over the sizes of its
parts: two relations, the last size below one wave and one workgroup of
subsets, the largest, the first beyond; and costs that overflow to infinity
(there and on the larger queries' paths), where only the left set decides."""
import numpy as np
import pytest

import oracle
from paper_2202_13511_amd import mpdp, workloads as W

from test_gpu_parity import CMS, check_memo, check_plan, check_stats, run_ws

pytestmark = pytest.mark.gpu


def shapes(n):
    yield W.star(n, n)
    yield W.random_tree(n, n + 1)
    if n >= 3:
        yield W.cycle(n, n)
        yield W.clique(n, n)
        yield W.random_connected(n, n, 0.3)
        yield W.all_equal_clique(n)


@pytest.mark.parametrize("cm", CMS)
@pytest.mark.parametrize("n", [2, 3, 5, 6, 7, 10, 11, 12, 13])
def test_sizes(n, cm):
    for q in shapes(n):
        res, gm = run_ws(q, cm)
        ref = oracle.mpdp(q, cm)
        check_memo(q, gm, ref)
        check_plan(q, res, ref)
        check_stats(q, res, ref, general=q.m != n - 1)
        if n <= 12:
            one = mpdp.mpdp_optimize_noalloc(q, cm)
            assert one.plan == res.plan and one.cost == res.cost
            for key in ("connected_sets", "ccp_pairs", "evaluated_pairs", "candidates"):
                assert one.stats[key] == res.stats[key]


@pytest.mark.parametrize("cm", CMS)
@pytest.mark.parametrize("make", [W.star, W.random_tree, W.cycle, lambda n, s: W.random_connected(n, s, 0.3)],
                         ids=["star", "tree", "cycle", "random"])
@pytest.mark.parametrize("n", [8, 12, 14])
def test_infinite_costs(n, make, cm):
    q = make(n, 3)
    q.card = np.where(np.arange(n) % 3 == 1, 1e308, 10.0)
    q.sel = np.where(np.arange(q.m) % 4 == 3, 1e-300, 1.0)
    res, gm = run_ws(q, cm)
    ref = oracle.mpdp(q, cm)
    assert np.isinf(ref.root_cost)
    check_memo(q, gm, ref)
    check_plan(q, res, ref)


@pytest.mark.parametrize("n", [2, 12, 13])
def test_levels_evaluated(n):
    """eval_launches counts the levels, however many share a launch."""
    for q in (W.star(n, 1), W.random_tree(n, 2)):
        for st in (run_ws(q, mpdp.MPDP_COST_COUT)[0].stats, mpdp.mpdp_optimize_noalloc(q, mpdp.MPDP_COST_COUT).stats):
            assert st["levels"] == st["eval_launches"] == n - 1
