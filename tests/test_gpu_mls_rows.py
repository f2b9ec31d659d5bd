"""Edges of the local search's kernels that keep the connection sums: block
counts on both sides of the 16- and 64-block forms (65: sums recomputed), rows
longer than what is kept of them, queues of one vertex and full ones, and edge
weights whose sums need 64 bits. Whole numbers: equal to the oracle."""
import numpy as np
import pytest

import graphgen
import oracle


def _heavy(g):
    # symmetric weights near 2^31: a few of them add up past 32 bits
    src = np.repeat(np.arange(len(g["xadj"]) - 1), np.diff(g["xadj"]))
    dst = g["adjncy"]
    w = (2 ** 31 - 1 - (src + dst) % 7).astype(np.int32)
    return dict(g, adjwgt=w)


GRAPHS = {
    "rgg": lambda: graphgen.rgg2d(6000, 9),
    "heavy": lambda: _heavy(graphgen.grid3d(16, 15, 14, seed=1, wmax=3)),
    "hubs": lambda: graphgen.rmat(13, 16),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("k,batch,queue", [(16, 1024, 64), (17, 64, 63), (64, 1024, 64), (65, 256, 64), (3, 512, 1)])
def test_kept_sums_match_oracle(name, k, batch, queue):
    import torch
    import paper_1710_08231_amd as gp
    g = GRAPHS[name]()
    part, res = oracle.partition(g, k, 0.05)
    want, ost = oracle.mls(g, part, k, res["lmax"], seed=3, global_iters=2, batch=batch, max_queue=queue)
    got, st = gp.mls_refine(gp.to_device(g), torch.from_numpy(part).cuda(), k, res["lmax"], seed=3, global_iters=2,
                            batch=batch, queue=queue)
    assert (st["gain"], st["searches"], st["moves"], st["local_iters"]) == \
           (ost["gain"], ost["searches"], ost["moves"], ost["local_iters"])
    assert np.array_equal(got.cpu().numpy(), want)
