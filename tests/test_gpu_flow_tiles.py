"""The training step of the learned proposal at the edges of its tiles: every number of slices that a
thread of the action gradient takes (N = 32 and 64 beside the sizes of test_gpu_flow), batches around the
16 paths of a tile, the 128 of a staged chunk and the 1024 threads of the loss weights.

Tolerances: the gradients as in test_gpu_flow (same bounds, same parameters). The loss from the log weights
themselves: (B + 16) roundings of 2^-53 on each of two sums of B terms, relative to the largest term of the
formula."""
import numpy as np
import pytest

import paper_1105_0542_amd as P
import test_gpu_flow as base

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = P.Context()
    yield c
    c.close()


@pytest.mark.parametrize("coefs,s,L", [(base.QUARTIC, 5, 4), (base.ODD, 6, 4)])
def test_gradient_at_two_and_four_slices_a_thread(ctx, coefs, s, L):
    base.test_gradient_matches_oracle(ctx, (coefs, 1.0, 0.0, 1.0, 1.0, s, 8, L, 0), 0.5)


@pytest.mark.parametrize("s", [1, 2, 7])
@pytest.mark.parametrize("B", [2, 15, 17, 129, 1023, 1025, 2600])
def test_loss_and_steps_at_batch_edges(ctx, s, B):
    beta = 0.3
    f = P.Flow(ctx, base.QUARTIC, 1.0, 0.0, 1.0, 1.0, 1 << s, 6, layers=4, batch=B, lr=0.0, beta=beta)
    whole = P.Flow(ctx, base.QUARTIC, 1.0, 0.0, 1.0, 1.0, 1 << s, 6, layers=4, batch=4096, lr=0.0, beta=beta)
    th = base._random_params(4, 5 + s)
    f.set_params(th)
    whole.set_params(th)
    loss, ell, g = f.grad(3, 50)
    assert np.array_equal(ell, whole.grad(3, 50)[1][:B])          # a path does not depend on the batch
    mx = 2.0 * ell.max()
    ref = (1 - beta) * (mx + np.log(np.mean(np.exp(2.0 * ell - mx)))) - beta * np.mean(ell)
    scale = max(1.0, abs(mx), np.abs(ell).max())
    assert abs(loss - ref) <= 4 * (B + 16) * 2.0 ** -53 * scale
    assert np.all(np.isfinite(g))
    losses, _ = f.train(3, 50, 3)                                 # lr = 0: the step counter alone moves
    assert losses[0] == loss
    assert losses[1] == f.grad(3, 51)[0] and losses[2] == f.grad(3, 52)[0]
    f.close()
    whole.close()
