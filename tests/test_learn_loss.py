"""CPU: the training loss over every number of channels a layer may end in, on the smallest lattices."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_0810_5365_amd import learn


@pytest.mark.parametrize("n", [1, 3])
@pytest.mark.parametrize("Vh", [8, 24, 40, 320])
@pytest.mark.parametrize("channels", [1, 2, 3, 4, 8])
def test_batch_loss_and_gradient(channels, Vh, n):
    """mean_i ||y_i - t_i||^2 / ||t_i||^2 and its gradient against float64.  Sums of N non-negative float32
    terms are off by at most N 2^-24 of themselves whatever their order (a term's own rounding included in
    N + 2); quotient and mean add a few more."""
    N = 12 * Vh * channels
    rng = np.random.default_rng(100 * channels + Vh + n)
    y, t = (rng.standard_normal(n * N).astype(np.float32) for _ in range(2))
    yt = torch.tensor(y, requires_grad=True)
    loss = learn.batch_loss(lambda x, g, k: x, SimpleNamespace(g=None), yt, torch.tensor(t), n)
    loss.backward()
    y64, t64 = y.astype(np.float64).reshape(n, N), t.astype(np.float64).reshape(n, N)
    tt = (t64 ** 2).sum(1)
    ref = (((y64 - t64) ** 2).sum(1) / tt).mean()
    grad = 2.0 * (y64 - t64) / tt[:, None] / n
    tol = 2 * (N + 8) * 2.0 ** -24
    assert abs(loss.item() - ref) <= tol * ref
    # beside those sums, the float32 difference itself: half an ulp of |y| + |t|
    err = np.abs(yt.grad.numpy().reshape(n, N) - grad)
    assert (err <= tol * np.abs(grad) + 2.0 ** -23 * (np.abs(y64) + np.abs(t64)) * 2.0 / tt[:, None] / n).all()
