"""The batched kernel where a batch is made of one kind of query: tiny ones."""
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
