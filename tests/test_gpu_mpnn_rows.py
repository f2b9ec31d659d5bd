"""GPU tests of the network's aggregation at every way a row is served: rows of
at most 192 entries by lanes (16 at a time), wider ones staged 256 neighbours at
a time and summed 32 and then one at a time. Inference equals the oracle bit for
bit; the gradient agrees with the binary64 reference."""
import numpy as np
import pytest

import graphgen
import oracle
from oracle import mpnn

pytestmark = pytest.mark.gpu

WIDTHS = [0, 1, 15, 16, 17, 31, 33, 63, 64, 65, 128, 129, 191, 192, 193, 255, 256, 257, 287, 288, 511, 512, 513, 545, 800]


def _graph(seed, weighted):
    """One hub of each width among 1,000 other vertices."""
    rng = np.random.default_rng(seed)
    n, edges = len(WIDTHS) + 1000, []
    for h, d in enumerate(WIDTHS):
        edges += [(h, int(v)) for v in len(WIDTHS) + rng.choice(1000, d, replace=False)]
    w = rng.integers(1, 60, len(edges)) if weighted else None
    return graphgen.from_edges(n, edges, weights=w, vwgt=rng.integers(1, 9, n) if weighted else None)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("k", [3, 16, 33, 64])
def test_rows_of_every_width(weighted, k):
    import torch
    import paper_1710_08231_amd as gp
    g = _graph(k, weighted)
    n = len(g["xadj"]) - 1
    rng = np.random.default_rng(k + 1)
    w = rng.normal(0, 0.25, oracle.mpnn_param_count(k)).astype(np.float32)
    dg, dw = gp.to_device(g), torch.from_numpy(w).cuda()
    Z, P = gp.mpnn_forward(dg, k, dw, seed=3)
    Zo, Po = oracle.mpnn_infer(g, k, w, seed=3)
    assert np.array_equal(Z.cpu().numpy(), Zo) and np.array_equal(P.cpu().numpy(), Po)
    t = rng.integers(0, k, n).astype(np.int32)
    grad, (edge, bal) = gp.mpnn_backward(dg, k, dw, torch.from_numpy(t).cuda(), seed=3, lam=0.7)
    wr = oracle.bf16(w).astype(np.float64)
    e64, b64, g64 = mpnn.loss_and_grad(g, k, wr, t, seed=3, lam=0.7)
    # binary32 sums of up to n * 64 products per entry: errors of a few 2^-24 of the largest entries
    assert abs(edge - e64) <= 1e-5 * abs(e64) and abs(bal - b64) <= 1e-5 * abs(b64) + 1e-9
    assert np.abs(grad.cpu().numpy() - g64).max() <= 1e-4 * np.abs(g64).max()
