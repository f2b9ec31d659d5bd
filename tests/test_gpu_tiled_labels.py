"""GPU tests of the admission by tiles with more than 256 labels against the
oracle's rounds: label counts on both sides of each variant (2,048, 8,192 and
12,288 labels) and of the rules that choose it (two vertices a label up to 2,048
labels, 64 above), with bounds that end every block's room in some tile and
loose ones, both direction settings, active sets, weights, and as a batch."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("x,y,z,k", [
    (26, 26, 25, 257), (26, 26, 25, 2048),  # 16,900 vertices
    (52, 51, 50, 2049), (51, 51, 50, 2049),  # 132,600 and 130,050: on both sides of 64 a label
    (81, 81, 80, 8192), (81, 81, 80, 8193), (93, 93, 91, 12288), (93, 93, 91, 12289)])
def test_refine(x, y, z, k):
    import torch
    import paper_1710_08231_amd as gp
    n = x * y * z
    rng = np.random.default_rng(k)
    g = graphgen.grid3d(x, y, z, seed=3, wmax=10)
    g["vwgt"] = rng.integers(1, 6, n).astype(np.int32)
    part = (np.arange(n, dtype=np.int64) * k // n).astype(np.int32)
    stray = rng.random(n) < 0.3
    part[stray] = rng.integers(0, k, int(stray.sum()))
    B = np.bincount(part, weights=g["vwgt"], minlength=k).astype(np.int64)
    dg, dp = gp.to_device(g), torch.from_numpy(part).cuda()
    for lm in (int(B.mean() * 1.05) + 5, int(B.max()) + 20):
        want, ost = oracle.lp_refine(g, part, k, lm, 4)
        got, st = gp.lp_refine(dg, dp, k, lm, 4)
        assert np.array_equal(got.cpu().numpy(), want)
        assert (st["rounds_run"], st["moves"]) == (ost["rounds_run"], ost["moves"])


@pytest.mark.parametrize("n", [520, 4096, 4097, 9000])
@pytest.mark.parametrize("k", [257, 259, 260, 261])
@pytest.mark.parametrize("alternate", [1, 0])
def test_active_refine_small(n, k, alternate):
    # at most 16,384 vertices only active sets (and batches) come here; 520 is two vertices a label at k = 260
    import torch
    import paper_1710_08231_amd as gp
    rng = np.random.default_rng(n + k)
    g = graphgen.rgg2d(n, 5)
    part = rng.integers(0, k, n).astype(np.int32)
    lm = int(np.bincount(part, minlength=k).mean() * 1.2) + 1
    want, ost = oracle.lp_refine(g, part, k, lm, 12, alternate, active=True)
    got, st = gp.lp_refine(gp.to_device(g), torch.from_numpy(part).cuda(), k, lm, 12, alternate, active=True)
    assert np.array_equal(got.cpu().numpy(), want)
    assert (st["rounds_run"], st["moves"], st["edge_visits"]) == (ost["rounds_run"], ost["moves"], ost["edge_visits"])


@pytest.mark.parametrize("count,n,k", [(150, 70, 2), (300, 150, 7), (40, 2500, 16)])
def test_batch(count, n, k):
    import paper_1710_08231_amd as gp
    gs = [graphgen.rgg2d(n + 3 * i, i) for i in range(count)]
    u, off = gp.union_graph(gs)
    part, res, _ = gp.partition_batch(gp.to_device(u), off, [k] * count, 0.03)
    part = part.cpu().numpy()
    for i in range(0, count, 7):
        assert np.array_equal(part[off[i]:off[i + 1]], oracle.partition(gs[i], k, 0.03)[0])
