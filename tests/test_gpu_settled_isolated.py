"""GPU tests of refinement on small levels with vertices without neighbours:
they are never evaluated, so they must not count as vertices left to evaluate
when the later rounds run in one launch. Thousands of them, with weights; the
kernel launches of a call are counted, and the result compared with the oracle's."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _with_isolated(n, iso, seed):
    """An rgg of n vertices whose ids are spread among n + iso, the others without neighbours."""
    g = graphgen.rgg2d(n, seed)
    rng = np.random.default_rng(seed)
    ids = np.sort(rng.permutation(n + iso)[:n])
    deg = np.zeros(n + iso, np.int64)
    deg[ids] = np.diff(g["xadj"])
    return {"xadj": np.concatenate([[0], np.cumsum(deg)]).astype(np.int32),
            "adjncy": ids[g["adjncy"]].astype(np.int32), "adjwgt": g.get("adjwgt"),
            "vwgt": rng.integers(1, 5, n + iso).astype(np.int32)}, ids


def _launches(call):
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        out = call()
        torch.cuda.synchronize()
    return out, sum(e.name == "hipLaunchKernel" for e in prof.events())


@pytest.mark.parametrize("k,n,iso", [(8, 600, 2049), (8, 600, 12000), (40, 500, 1500)])
@pytest.mark.parametrize("alternate", [1, 0])
def test_isolated_vertices_are_not_evaluated(k, n, iso, alternate):
    import torch
    import paper_1710_08231_amd as gp
    g, ids = _with_isolated(n, iso, 3)
    part = np.random.default_rng(k).integers(0, k, n + iso).astype(np.int32)
    part[ids] = np.arange(n) * k // n
    part[ids[::9]] = 0
    W = np.bincount(part, weights=g["vwgt"], minlength=k).astype(np.int64)
    lm = int(W.max() * 1.05)
    P, moves, idle, r = part.copy(), 0, 0, 0
    while r < 25 and idle < 2:
        P, W, m, _ = oracle.lp_round(g, P, W, lm, r, alternate)
        idle = idle + 1 if m == 0 else 0
        moves += m
        r += 1
    assert r > 10
    dg, dp = gp.to_device(g), torch.from_numpy(part).cuda()
    _, two = _launches(lambda: gp.lp_refine(dg, dp, k, lm, 2, dir_alternate=alternate))
    (got, st), all_rounds = _launches(lambda: gp.lp_refine(dg, dp, k, lm, 25, dir_alternate=alternate))
    assert np.array_equal(got.cpu().numpy(), P)
    assert (st["rounds_run"], st["moves"]) == (r, moves)
    # two rounds launched as before, the vertices to evaluate set, the other rounds: at most two launches more
    assert 0 < two < all_rounds <= two + 2
