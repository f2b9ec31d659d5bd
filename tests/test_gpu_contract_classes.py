"""Edges of the contraction's row classes: coarse rows of 1, 15 to 17, 31 to 33,
127 to 129, 511 to 513 and 2047 to 2049 fine entries, from one member and from
many, with and without weights. Equal to the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

SIZES = (1, 15, 16, 17, 31, 32, 33, 127, 128, 129, 511, 512, 513, 2047, 2048, 2049)


def _stars(split, weighted, seed):
    # one coarse row per size: `split` members that share the row's entries, to leaves of few labels
    rng = np.random.default_rng(seed)
    edges, w, labels = [], [], []
    leaves = 4200
    labels = list(range(leaves))
    nv = leaves
    for r, d in enumerate(SIZES):
        m = min(split, d)
        ends = rng.permutation(leaves)[:d]
        for q in range(m):
            labels.append(leaves + r)
            for x in ends[q::m]:
                edges.append((nv, int(x)))
                w.append(int(rng.integers(1, 2 ** 20)))
            nv += 1
    labels = np.array(labels, np.int32)
    labels[:leaves] = labels[:leaves] // 3  # leaves share columns
    g = graphgen.from_edges(nv, edges, weights=w if weighted else None)
    return g, labels


@pytest.mark.gpu
@pytest.mark.parametrize("split", [1, 5, 40])
@pytest.mark.parametrize("weighted", [False, True])
def test_row_classes_match_oracle(split, weighted):
    import torch
    import paper_1710_08231_amd as gp
    g, labels = _stars(split, weighted, 3)
    ocg, of2c = oracle.contract(g, labels)
    cg, f2c = gp.contract(gp.to_device(g), torch.from_numpy(labels).cuda())
    assert np.array_equal(f2c.cpu().numpy(), of2c)
    for key in ("xadj", "adjncy", "adjwgt", "vwgt"):
        assert np.array_equal(cg[key].cpu().numpy(), ocg[key]), key
