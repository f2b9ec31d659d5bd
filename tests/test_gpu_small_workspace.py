"""GPU tests of the scratch of small calls: a workspace that once was enough for a
call (as it was reported before the admission's buffers changed) still is."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _graph(kind, n):
    return graphgen.rgg2d(n, 3) if kind == "rgg" else graphgen.from_edges(n, [(0, i) for i in range(1, n)])


def _ws(size):
    import torch
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    assert ws.data_ptr() % 256 == 0
    return ws


@pytest.mark.parametrize("kind,n,active,size", [("rgg", 60, False, 5632), ("star", 60, True, 8704),
                                                ("star", 1000, True, 70144)])
def test_cluster(kind, n, active, size):
    import paper_1710_08231_amd as gp
    g = _graph(kind, n)
    U = max(2, n // 20)
    lab, st = gp.lp_cluster(gp.to_device(g), U, 10, active=active, ws=_ws(size))
    want = oracle.lp_cluster(g, U, 10, active=active)[0]
    assert np.array_equal(lab.cpu().numpy(), want) and st["workspace_bytes"] <= size


@pytest.mark.parametrize("kind,n,k,active,size", [
    ("rgg", 2, 256, True, 9728), ("rgg", 100, 2, False, 8704), ("rgg", 100, 256, True, 13312),
    ("star", 200, 16, False, 14592), ("star", 200, 256, True, 22528), ("star", 300, 300, True, 24320), ("rgg", 455, 64, True, 44800),
    ("rgg", 1000, 300, True, 61952)])
def test_refine(kind, n, k, active, size):
    import torch
    import paper_1710_08231_amd as gp
    g = _graph(kind, n)
    part = (np.arange(n) % k).astype(np.int32)
    for lm in (2 * n, -(-n // k) + 1):
        want = oracle.lp_refine(g, part, k, lm, 25, active=active)[0]
        for ws in (_ws(size), None):  # without one also with connection rows
            got, st = gp.lp_refine(gp.to_device(g), torch.from_numpy(part).cuda(), k, lm, 25, active=active, ws=ws)
            assert np.array_equal(got.cpu().numpy(), want)
            assert ws is None or st["workspace_bytes"] <= size


@pytest.mark.parametrize("n,k,size", [(60, 16, 50688), (300, 2, 77568)])
def test_partition(n, k, size):
    import paper_1710_08231_amd as gp
    g = graphgen.rgg2d(n, 3)
    part, res = gp.partition(gp.to_device(g), k, 0.03, ws=_ws(size))
    assert np.array_equal(part.cpu().numpy(), oracle.partition(g, k, 0.03)[0]) and res["workspace_bytes"] <= size


def test_partition_batch():
    import paper_1710_08231_amd as gp
    gs = [graphgen.rgg2d(50, s) for s in range(2)]
    u, off = gp.union_graph(gs)
    part, _, _ = gp.partition_batch(gp.to_device(u), off, [2, 2], 0.03, ws=_ws(49408))
    want = np.concatenate([oracle.partition(g, 2, 0.03)[0] for g in gs])
    assert np.array_equal(part.cpu().numpy(), want)


@pytest.mark.parametrize("k,size", [(8192, 159734528), (12288, 159783680), (12289, 159784192)])
def test_refine_with_many_blocks(k, size):
    # the label sums of the tiled admission are largest here
    import torch
    import paper_1710_08231_amd as gp
    g = graphgen.rmat(20, 3)
    n = len(g["xadj"]) - 1
    part = (np.arange(n, dtype=np.int64) * k // n).astype(np.int32)
    part[::5] = np.random.default_rng(k).integers(0, k, len(part[::5]))
    lm = 2 * n // k + 2
    want, _ = oracle.lp_refine(g, part, k, lm, 2)
    got, st = gp.lp_refine(gp.to_device(g), torch.from_numpy(part).cuda(), k, lm, 2, ws=_ws(size))
    assert np.array_equal(got.cpu().numpy(), want) and st["workspace_bytes"] <= size
