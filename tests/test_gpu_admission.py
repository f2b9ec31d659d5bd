"""GPU tests of the admission kernels against the oracle's rounds.

The proposers to a target are admitted in ascending id while they fit. Up to
256 labels the GPU works on tiles of 4,096 vertices and finds the one in which
a target's room ends; with more labels it works on tiles of 2,048, moves the
proposers of targets with room for all at once, and selects among the others
per target (up to 64 proposers in one wave, more by a radix selection over
ids). Sizes on both sides of a tile, targets with few and many proposers, room
ending at once, in the middle and nowhere, unit and mixed weights.
"""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _hubs(n, fan, seed, weighted):
    """Groups of `fan` consecutive vertices around a hub each, hubs joined in a ring: every leaf
    proposes its hub's label, so a target has about `fan` proposers."""
    rng = np.random.default_rng(seed)
    hub = np.arange(n) // (fan + 1) * (fan + 1)
    edges = [(int(h), int(v)) for v, h in enumerate(hub) if v != h]
    heads = np.unique(hub)
    edges += [(int(a), int(b)) for a, b in zip(heads[:-1], heads[1:])]
    g = graphgen.from_edges(n, edges, weights=rng.integers(1, 9, len(edges)) if weighted else None,
                            vwgt=rng.integers(1, 6, n) if weighted else None)
    return g


@pytest.mark.parametrize("n", [16385, 18431, 18432, 18433, 20480])
@pytest.mark.parametrize("fan", [3, 63, 64, 65, 700])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("share", [0.02, 0.6, 4.0])
def test_cluster_admission(n, fan, weighted, share):
    import paper_1710_08231_amd as gp
    g = _hubs(n, fan, 3, weighted)
    U = max(6, int(share * fan * (3 if weighted else 1)))
    for alternate in (1, 0):
        lab, st = gp.lp_cluster(gp.to_device(g), U, 6, dir_alternate=alternate)
        want, ost = _cluster(g, U, 6, alternate)
        assert np.array_equal(lab.cpu().numpy(), want)
        assert (st["rounds_run"], st["moves"]) == ost


def _cluster(g, U, rounds, alternate):
    if alternate:
        lab, st = oracle.lp_cluster(g, U, rounds)
        return lab, (st["rounds_run"], st["moves"])
    n = len(g["xadj"]) - 1
    C, W = np.arange(n, dtype=np.int32), np.ones(n, np.int64) if g.get("vwgt") is None else g["vwgt"].astype(np.int64)
    moves, idle, r = 0, 0, 0
    while r < rounds and idle < 2:
        C, W, m, _ = oracle.lp_round(g, C, W, U, r, 0)
        idle = idle + 1 if m == 0 else 0
        moves += m
        r += 1
    return C, (r, moves)


@pytest.mark.parametrize("n", [16385, 20479, 20480, 20481])
@pytest.mark.parametrize("k", [2, 17, 256, 257, 400])
@pytest.mark.parametrize("weighted", [False, True])
def test_refine_admission(n, k, weighted):
    # blocks at, just below and far below their bound
    import torch
    import paper_1710_08231_amd as gp
    rng = np.random.default_rng(n + k)
    g = graphgen.rgg2d(n, 5)
    if weighted:
        g["vwgt"] = rng.integers(1, 9, n).astype(np.int32)
    part = rng.integers(0, k, n).astype(np.int32)
    B = np.bincount(part, weights=g.get("vwgt"), minlength=k).astype(np.int64)
    for lm in (int(B.max()), int(B.mean() * 1.2) + 9, int(B.sum())):
        want, ost = oracle.lp_refine(g, part, k, lm, 8)
        for call in (gp.lp_refine, gp.lp_refine_static):
            got, st = call(gp.to_device(g), torch.from_numpy(part).cuda(), k, lm, 8)
            assert np.array_equal(got.cpu().numpy(), want)
            assert (st["rounds_run"], st["moves"]) == (ost["rounds_run"], ost["moves"])


@pytest.mark.parametrize("k", [5, 64, 300])
@pytest.mark.parametrize("alternate", [1, 0])
def test_settled_vertices_on_hub_graphs(k, alternate):
    # vertices without a better block are not evaluated again until a neighbour moves; here hubs far
    # above 256 neighbours move too (tight and loose bounds, with connection rows and without)
    import torch
    import paper_1710_08231_amd as gp
    g = graphgen.rmat(15, 8)
    n = len(g["xadj"]) - 1
    rng = np.random.default_rng(k)
    part = rng.integers(0, k, n).astype(np.int32)
    B = np.bincount(part, minlength=k).astype(np.int64)
    for lm in (int(B.max()), 2 * n):
        P, W, moves, idle, r = part.copy(), B.copy(), 0, 0, 0
        while r < 25 and idle < 2:
            P, W, m, _ = oracle.lp_round(g, P, W, lm, r, alternate)
            idle = idle + 1 if m == 0 else 0
            moves += m
            r += 1
        for call in (gp.lp_refine, gp.lp_refine_static):
            got, st = call(gp.to_device(g), torch.from_numpy(part).cuda(), k, lm, 25, dir_alternate=alternate)
            assert np.array_equal(got.cpu().numpy(), P)
            assert (st["rounds_run"], st["moves"]) == (r, moves)
