"""GPU tests of refinement on small levels: after two launched rounds one
workgroup runs all later rounds in one launch, unless more than 2,048 vertices
have to be evaluated at once (the launched rounds go on then). Against the
oracle's rounds, both outcomes, every table width, weights, both direction
settings, sizes around the limits (16,384 vertices)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _rounds(g, part, k, lm, rounds, alternate):
    w = g.get("vwgt")
    P, W = part.copy(), np.bincount(part, weights=w, minlength=k).astype(np.int64)
    moves, idle, r = 0, 0, 0
    while r < rounds and idle < 2:
        P, W, m, _ = oracle.lp_round(g, P, W, lm, r, alternate)
        idle = idle + 1 if m == 0 else 0
        moves += m
        r += 1
    return P, (r, moves)


@pytest.mark.parametrize("n", [200, 2049, 4096, 16383, 16384])
@pytest.mark.parametrize("k", [2, 16, 17, 50])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("start", ["stripes", "random"])
def test_refine_small(n, k, weighted, start):
    import torch
    import paper_1710_08231_amd as gp
    rng = np.random.default_rng(n * k)
    g = graphgen.rgg2d(n, 7)
    if weighted:
        g["vwgt"] = rng.integers(1, 9, n).astype(np.int32)
        deg = np.diff(g["xadj"])
        src = np.repeat(np.arange(n), deg)
        g["adjwgt"] = (1 + (np.minimum(src, g["adjncy"]) * 7 + np.maximum(src, g["adjncy"])) % 9).astype(np.int32)
    part = (np.arange(n) * k // n).astype(np.int32)
    if start == "random":  # most vertices stay unsettled for a while
        part = rng.integers(0, k, n).astype(np.int32)
    else:
        stray = rng.random(n) < 0.1
        part[stray] = rng.integers(0, k, int(stray.sum()))
    B = np.bincount(part, weights=g.get("vwgt"), minlength=k).astype(np.int64)
    for lm in (int(B.max()), int(1.1 * B.max()), int(B.sum())):
        for alternate in (1, 0):
            want, counts = _rounds(g, part, k, lm, 25, alternate)
            for call in (gp.lp_refine, gp.lp_refine_static):
                got, st = call(gp.to_device(g), torch.from_numpy(part).cuda(), k, lm, 25, dir_alternate=alternate)
                assert np.array_equal(got.cpu().numpy(), want)
                assert (st["rounds_run"], st["moves"]) == counts


@pytest.mark.parametrize("k", [100, 256, 1100, 5000])
@pytest.mark.parametrize("rounds", [1, 2, 3, 25])
def test_refine_small_many_blocks(k, rounds):
    # tables of 256 sums, label weights in and out of LDS, more blocks than fit the small round's sums
    import torch
    import paper_1710_08231_amd as gp
    rng = np.random.default_rng(k)
    for n in (3000, 16384):
        g = graphgen.rmat_m(14, 60000, 5) if n == 16384 else graphgen.rgg2d(n, 9)
        part = rng.integers(0, k, n).astype(np.int32)
        lm = int(np.bincount(part, minlength=k).max())
        want, counts = _rounds(g, part, k, lm, rounds, 1)
        got, st = gp.lp_refine(gp.to_device(g), torch.from_numpy(part).cuda(), k, lm, rounds)
        assert np.array_equal(got.cpu().numpy(), want) and (st["rounds_run"], st["moves"]) == counts
