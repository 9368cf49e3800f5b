"""A workspace sized for n relations serves every smaller query."""
import numpy as np
import pytest

from paper_2202_13511_amd import mpdp, workloads as W


def test_workspace_never_shrinks():
    sizes = [mpdp.mpdp_workspace_bytes(n) for n in range(1, 33)]
    assert sizes == sorted(sizes)
    assert mpdp.mpdp_workspace_bytes(0) == mpdp.mpdp_workspace_bytes(33) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("n", [17, 18, 19])
def test_smaller_query_in_a_workspace_for_19(n):
    q = W.cycle_chords(3, n=n, chords=4)
    ws = mpdp.workspace(19)
    got = mpdp.mpdp_optimize_ws(q, mpdp.MPDP_COST_PGLIKE, ws)
    assert got.plan == mpdp.mpdp_optimize(q, mpdp.MPDP_COST_PGLIKE).plan
    assert np.isfinite(got.cost)
