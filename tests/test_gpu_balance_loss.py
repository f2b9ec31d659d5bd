"""GPU test of the balance term of the training loss: it is the difference of a
block's share of the weight and 1 / k, so its sums are binary64. Calls on the
same inputs agree to the order of those sums, whichever lane comes first, and
with the term of the binary64 reference."""
import numpy as np
import pytest

import graphgen
import oracle
from oracle import mpnn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 33, 64])
@pytest.mark.parametrize("n", [7, 813, 2500])
def test_balance_loss_repeats(k, n):
    import torch
    import paper_1710_08231_amd as gp
    rng = np.random.default_rng(n + k)
    g = graphgen.rgg2d(n, 5)
    g["vwgt"] = rng.integers(1, 41, n).astype(np.int32)
    w = rng.normal(0, 0.15, oracle.mpnn_param_count(k)).astype(np.float32)
    t = rng.integers(0, k, n).astype(np.int32)
    dg, dw, dt = gp.to_device(g), torch.from_numpy(w).cuda(), torch.from_numpy(t).cuda()
    bal = [gp.mpnn_backward(dg, k, dw, dt, seed=3, lam=0.7)[1][1] for _ in range(8)]
    # the shares are sums of n binary64 products: their error is below n 2^-53, and the term's derivative by
    # a share is 2 lam k |share - 1 / k| <= 2 lam k sqrt(term / (lam k)); k shares
    tol = 2 * k * n * 2.0 ** -53 * np.sqrt(0.7 * k * max(bal)) + 1e-25
    assert max(bal) - min(bal) <= tol
    _, b64, _ = mpnn.loss_and_grad(g, k, oracle.bf16(w).astype(np.float64), t, seed=3, lam=0.7)
    # binary32 logits and probabilities, 2^-18 at most of each share
    assert abs(bal[0] - b64) <= 2 * 2.0 ** -18 * np.sqrt(0.7 * k * b64) + 2.0 ** -36 * 0.7 * k
