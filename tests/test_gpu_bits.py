"""Cyclic queries that test every subset against a connectivity bitmap: at the
edges of its range (one launch below, lists above), sparse and dense, with
ties, with costs beyond the largest double.  Cost, plan and counters against
the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2202_13511_amd import mpdp
from paper_2202_13511_amd import workloads as W

pytestmark = pytest.mark.gpu


def tied(n):
    q = W.cycle_chords(n, n=n, chords=4)
    q.card[:] = 1000.0
    q.sel[:] = 0.001
    return q


def huge(n):
    q = W.random_connected(n, n, extra=0.2)
    q.card[:] = 1e308
    q.sel[:] = 1.0
    return q


CASES = [W.cycle(13, 1), W.random_connected(13, 2, extra=0.3), W.clique(13, 3), W.all_equal_clique(13),
         W.cycle_chords(5, n=14, chords=2), W.random_connected(15, 6, extra=0.15), tied(16), huge(13),
         W.cycle_chords(7, n=17, chords=6), W.cycle_chords(8, n=18, chords=3), W.cycle_chords(9, n=19, chords=2)]


@pytest.mark.parametrize("cm", [mpdp.MPDP_COST_COUT, mpdp.MPDP_COST_PGLIKE])
@pytest.mark.parametrize("q", CASES, ids=lambda q: f"{q.name}-{q.n}")
def test_matches_oracle(q, cm):
    ref = oracle.mpdp(q, cm)
    want = oracle.plan_from_memo(ref)
    ws = mpdp.workspace(q.n, cm)
    for flags in (0, mpdp.MPDP_FLAG_TIMING):
        got = mpdp.mpdp_optimize_ws(q, cm, ws, flags=flags)
        assert np.float64(got.cost).view(np.uint64) == np.float64(ref.root_cost).view(np.uint64)
        assert [(p["relset"], p["left"], p["right"], p["op"]) for p in got.plan] == \
               [(p["relset"], p["left"], p["right"], p["op"]) for p in want]
        assert got.stats["connected_sets"] == ref.connected_sets
        assert got.stats["ccp_pairs"] == ref.ccp_ordered // 2
        assert got.stats["evaluated_pairs"] == ref.evaluated
