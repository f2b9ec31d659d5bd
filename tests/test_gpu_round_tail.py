"""GPU tests of the one-workgroup round tail (at most 16,384 vertices) against the
oracle: both thread shapes (4 and 16 vertices a thread: up to 4,096 vertices and
labels, above), rounds that refuse proposals before and after rounds that refuse
none, one target for nearly all proposers (a star), and the rules of the settled
rounds that follow it (eight rounds, at most 32 neighbours a vertex)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _graph(kind, n):
    if kind == "star":
        return graphgen.from_edges(n, [(0, i) for i in range(1, n)])
    if kind == "dense":  # above 32 neighbours a vertex
        return graphgen.random_small(min(n, 700), 0.15, 9, wmax=9, vmax=5)
    return graphgen.rgg2d(n, 5)


@pytest.mark.parametrize("kind,n", [("rgg", 65), ("rgg", 1025), ("rgg", 4095), ("rgg", 4096), ("rgg", 4097),
                                    ("rgg", 16384), ("star", 300), ("star", 4096), ("star", 16384), ("dense", 700)])
@pytest.mark.parametrize("k", [2, 16, 33, 300])
def test_refine(kind, n, k):
    import torch
    import paper_1710_08231_amd as gp
    rng = np.random.default_rng(n + k)
    g = _graph(kind, n)
    part = rng.integers(0, k, n).astype(np.int32)
    w = g.get("vwgt")
    B = np.bincount(part, weights=w, minlength=k).astype(np.int64)
    dg, dp = gp.to_device(g), torch.from_numpy(part).cuda()
    for lm in (int(B.max()), int(B.mean() * 1.3) + 6, int(B.sum())):
        for rounds in (1, 7, 8, 25):
            want, ost = oracle.lp_refine(g, part, k, lm, rounds)
            got, st = gp.lp_refine(dg, dp, k, lm, rounds)
            assert np.array_equal(got.cpu().numpy(), want)
            assert (st["rounds_run"], st["moves"]) == (ost["rounds_run"], ost["moves"])


@pytest.mark.parametrize("n,k", [(3000, 4096), (3000, 4097), (4096, 16384), (60, 5000)])
def test_more_labels_than_the_small_shape_holds(n, k):
    import torch
    import paper_1710_08231_amd as gp
    rng = np.random.default_rng(k)
    g = graphgen.rgg2d(n, 7)
    part = rng.integers(0, k, n).astype(np.int32)
    for lm in (1, 2, n):
        want, ost = oracle.lp_refine(g, part, k, lm, 9)
        got, st = gp.lp_refine(gp.to_device(g), torch.from_numpy(part).cuda(), k, lm, 9)
        assert np.array_equal(got.cpu().numpy(), want) and st["moves"] == ost["moves"]


@pytest.mark.parametrize("kind,n", [("rgg", 4096), ("rgg", 4097), ("rgg", 16384), ("star", 4097), ("dense", 700)])
def test_cluster(kind, n):
    import paper_1710_08231_amd as gp
    g = _graph(kind, n)
    for U in (6, 40, 5 * n):
        want, ost = oracle.lp_cluster(g, U, 10)
        got, st = gp.lp_cluster(gp.to_device(g), U, 10)
        assert np.array_equal(got.cpu().numpy(), want)
        assert (st["rounds_run"], st["moves"]) == (ost["rounds_run"], ost["moves"])
