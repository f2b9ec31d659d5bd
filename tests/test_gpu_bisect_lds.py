"""Edges of the bisection kernels: graphs at and above the size whose marks are
kept in LDS (4096 vertices), few and many workgroups (512 of 1024 threads fit
the chip), frontiers with more edges than a thread keeps between its passes,
and subproblems of several components. Equal to the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

GRAPHS = {
    "below": lambda: graphgen.rgg2d(4095, 2),
    "at": lambda: graphgen.rgg2d(4096, 3),
    "above": lambda: graphgen.rgg2d(4097, 4),
    "dense": lambda: graphgen.rmat(9, 64),
    "parts": lambda: graphgen.rgg2d(700, 5),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("k,attempts", [(2, 1), (16, 5), (128, 16)])
def test_bisection_matches_oracle(name, k, attempts):
    import paper_1710_08231_amd as gp
    g = GRAPHS[name]()
    # every vertex count above is at or below the coarsest size for large k: few or no levels before the bisections
    want, ores = oracle.partition(g, k, 0.05, attempts=attempts, seed=7)
    got, res = gp.partition(gp.to_device(g), k, 0.05, attempts=attempts, seed=7)
    assert np.array_equal(got.cpu().numpy(), want) and res["cut"] == ores["cut"]


@pytest.mark.gpu
@pytest.mark.parametrize("count", [40, 300])
def test_batched_bisections_match_single(count):
    import paper_1710_08231_amd as gp
    gs = [graphgen.rgg2d(120 + 37 * (i % 11), i) for i in range(count)]
    u, off = gp.union_graph(gs)
    ks = [4 + 4 * (i % 2) for i in range(count)]
    part, _, _ = gp.partition_batch(gp.to_device(u), off, ks, 0.05, seed=5)
    part = part.cpu().numpy()
    for i in (0, 1, count // 2, count - 1):
        want, _ = oracle.partition(gs[i], ks[i], 0.05, seed=5)
        assert np.array_equal(part[off[i]:off[i + 1]], want)
