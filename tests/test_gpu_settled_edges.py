"""GPU tests at the edges of two rules, against the oracle.

Later refinement rounds in one launch with 17 to 64 blocks: taken up to 2,048
vertices, given up while more than 1,024 are to be evaluated (up to 16 blocks:
2,048, tried again unless there are more than twice as many).

Labels gathered with the class of their room: the class is exact below 16 and has
eight steps per doubling above, so vertex weights and rooms lie around 16, around
powers of two and their eighths, above INT_MAX and below zero."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1024, 1025, 1100, 2047, 2048, 2049])
@pytest.mark.parametrize("k", [17, 50, 64])
@pytest.mark.parametrize("alternate", [1, 0])
def test_settled_rounds_up_to_64_blocks(n, k, alternate):
    import torch
    import paper_1710_08231_amd as gp
    rng = np.random.default_rng(n * k)
    g = graphgen.rgg2d(n, 7)
    assert len(g["adjncy"]) <= 32 * n
    part = rng.integers(0, k, n).astype(np.int32)  # nearly all vertices are to be evaluated at first
    for lm in (int(np.bincount(part, minlength=k).max()), n):
        want, ost = oracle.lp_refine(g, part, k, lm, 25, alternate)
        for call in (gp.lp_refine, gp.lp_refine_static):
            got, st = call(gp.to_device(g), torch.from_numpy(part).cuda(), k, lm, 25, dir_alternate=alternate)
            assert np.array_equal(got.cpu().numpy(), want)
            assert (st["rounds_run"], st["moves"]) == (ost["rounds_run"], ost["moves"])


@pytest.mark.parametrize("k", [3, 16])
@pytest.mark.parametrize("live", [1900, 2100, 4000, 4400, 9000])
def test_tries_up_to_16_blocks(k, live):
    # about `live` scattered vertices of 16,000: one try, several tries, none after the first
    import torch
    import paper_1710_08231_amd as gp
    rng = np.random.default_rng(live)
    g = graphgen.grid3d(25, 25, 25, seed=1, wmax=10)
    n = 25 ** 3
    part = (np.arange(n) * k // n).astype(np.int32)
    stray = rng.permutation(n)[:live // 3]
    part[stray] = rng.integers(0, k, len(stray))
    lm = int(np.bincount(part, minlength=k).max())
    want, ost = oracle.lp_refine(g, part, k, lm, 25)
    got, st = gp.lp_refine(gp.to_device(g), torch.from_numpy(part).cuda(), k, lm, 25)
    assert np.array_equal(got.cpu().numpy(), want)
    assert (st["rounds_run"], st["moves"]) == (ost["rounds_run"], ost["moves"])


STEPS = [1, 2, 7, 8, 14, 15, 16, 17, 18, 19, 31, 32, 33, 35, 36, 255, 256, 257, 287, 288, 289]


@pytest.mark.parametrize("weights,bounds", [
    (STEPS, [15, 16, 17, 33, 48, 289, 300, 575, 1024]),  # some vertices are heavier than the bound: room below zero
    ([1 << 20, (1 << 20) + 1, (1 << 23) - 1, 1 << 23], [(1 << 23) + 5, 1 << 24, (1 << 31) - 1, (1 << 31) + 9, 1 << 40]),
    ([1, (1 << 30) + 1, (1 << 31) - 1], [(1 << 31) - 1, 1 << 31, (1 << 32) + 3, 1 << 50])])
@pytest.mark.parametrize("alternate", [1, 0])
def test_room_classes(weights, bounds, alternate):
    import paper_1710_08231_amd as gp
    g = graphgen.rmat(15, 8)
    n = len(g["xadj"]) - 1
    deg = np.diff(g["xadj"])
    assert n > 16384 and deg[deg > 64].sum() >= 4 * n  # the wide tiers gather four labels a vertex
    g["vwgt"] = np.random.default_rng(n).choice(weights, n).astype(np.int32)
    dg = gp.to_device(g)
    for U in bounds:
        want, ost = oracle.lp_cluster(g, U, 6, alternate)
        got, st = gp.lp_cluster(dg, U, 6, dir_alternate=alternate)
        assert np.array_equal(got.cpu().numpy(), want), U
        assert (st["rounds_run"], st["moves"]) == (ost["rounds_run"], ost["moves"])
