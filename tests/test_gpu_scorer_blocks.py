"""The scorer's kernels at the edges of their blocks (32 batch rows forward,
16-row matrix steps and fetches of 256 and 512 rows backward) and with inputs
and work buffers that are not aligned for 16-byte accesses, against
oracle/mlp.py with its own per-element bounds."""
import numpy as np
import pytest

from oracle import mlp
from paper_2202_13511_amd import mpdp

from test_gpu_scorer import grid_batch, grid_params, within

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 31, 33, 255, 256, 511, 512, 513, 1040])
def test_gradients_at_block_edges(B):
    w = grid_params(B)
    x, y = grid_batch(B, B)
    block = mpdp.scorer_params()
    mpdp.scorer_load(block, w)
    loss = mpdp.scorer_grad(block, x, y)
    want_loss, want = mlp.loss_and_grads(w, x, y)
    assert abs(loss - want_loss) <= 1e-5 * abs(want_loss) + 1e-6
    got = mpdp.scorer_grads(block)
    bounds = mlp.error_bounds(w, x, y)
    for k in want:
        within(got[k], want[k], bounds[k], k)


def test_unaligned_buffers_give_the_same_bits():
    import torch
    B = 77
    w = grid_params(1)
    x, y = grid_batch(2, B)
    xs = torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda()
    ys = torch.from_numpy(y).cuda()
    odd = torch.empty(B * 32 + 1, dtype=torch.int16, device="cuda")[1:].view(B, 32)
    odd.copy_(xs)
    work = mpdp.scorer_work(B)
    odd_work = torch.zeros(work.numel() + 4, dtype=torch.uint8, device="cuda")[4:]
    out = []
    for xx, ww in ((xs, work), (odd, work), (xs, odd_work), (odd, odd_work)):
        block = mpdp.scorer_params()
        mpdp.scorer_load(block, w)
        logits = mpdp.scorer_forward(block, xx, work=ww)
        mpdp.scorer_train_step(block, xx, ys, 1e-3, 1, work=ww)
        out.append((logits, mpdp.scorer_weights(block), mpdp.scorer_grads(block)))
    for o in out[1:]:
        assert np.array_equal(o[0], out[0][0])
        for k in w:
            assert np.array_equal(o[1][k], out[0][1][k]) and np.array_equal(o[2][k], out[0][2][k]), k
