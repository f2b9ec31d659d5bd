"""Edges of the contraction's row classes on graphs of more than 2^20 entries,
which use all of them (smaller ones use three): the stars of the small test
beside a grid whose pairs, runs of seven and one large cluster give rows of
every length between. Equal to the oracle."""
import numpy as np
import pytest

import graphgen
import oracle
from test_gpu_contract_classes import _stars

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", [1, 5, 40])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("group", [1, 2, 7, 60])
def test_row_classes_match_oracle(split, weighted, group):
    import torch
    import paper_1710_08231_amd as gp
    s, slab = _stars(split, weighted, 3)
    g = graphgen.grid3d(57, 56, 58, seed=2, wmax=10)
    if not weighted:
        g["adjwgt"] = None
    n = len(g["xadj"]) - 1
    u, off = gp.union_graph([s, g])
    assert len(u["adjncy"]) > 2 ** 20
    glab = np.arange(n) // group * group
    glab[-900:] = glab[-900]  # one row of the workgroup class
    labels = np.concatenate([slab, off[1] + glab]).astype(np.int32)
    ocg, of2c = oracle.contract(u, labels)
    cg, f2c = gp.contract(gp.to_device(u), torch.from_numpy(labels).cuda())
    assert np.array_equal(f2c.cpu().numpy(), of2c)
    for key in ("xadj", "adjncy", "adjwgt", "vwgt"):
        assert np.array_equal(cg[key].cpu().numpy(), ocg[key]), key
