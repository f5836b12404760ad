"""The traversal's settings (launch shape, list size, cell size) away from their
defaults: what the launches do differently, and the FP64 oracle's gradient."""
import numpy as np
import pytest
import torch

import oracle
from paper_2401_13708_amd import hts, synth
from gpu_inputs import embedding, rel

pytestmark = pytest.mark.gpu


@pytest.fixture
def settings(ctx):
    yield ctx
    ctx.set_item_points(hts.DEFAULT_ITEM_POINTS)
    ctx.set_item_list(hts.DEFAULT_ITEM_LIST)
    ctx.set_traversal_launch()


def _run(ctx, Y, csr):
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (Y, *csr)]
    tree = hts.Tree(ctx, Y.shape[0], 20)
    hts.build_polar_tree(ctx, dev[0], tree)
    st = torch.zeros(hts.STATS_PER_CALL, dtype=torch.int64, device="cuda")
    g, z = hts.gradient_bh(ctx, *dev, tree, 0.5, 12.0, stats=st)
    g2, z2 = hts.gradient_bh(ctx, *dev, tree, 0.5, 12.0)
    torch.cuda.synchronize()
    assert ctx.check() == 0
    tree.close()
    assert torch.equal(g, g2) and torch.equal(z, z2)
    return g, z, st


def _csr(n, dtype):
    return synth.random_csr(n, min(20, max(1, n // 4)), seed=3, dtype=dtype)


# waves that are whole sets of one for each part of the lists, and others
@pytest.mark.parametrize("n", [300, 13000])
def test_results_do_not_depend_on_the_launch_shape(settings, n):
    ctx = settings
    Y, csr = embedding(n, "late", np.float32), _csr(n, np.float32)
    want = _run(ctx, Y, csr)
    for shape in [(1, 1), (63, 1), (64, 1), (65, 2), (1000, 1), (1000, 4), (65537, 1)]:
        ctx.set_traversal_launch(*shape)
        for a, b in zip(_run(ctx, Y, csr), want):
            assert torch.equal(a, b), shape


# a wave whose share is full goes on without offering cells; the share fills with
# chunks (lists of 1 and 7) or with cells (small ones)
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("item_list,item_points", [(0, 288), (1, 288), (1, 3), (2, 20), (7, 288), (7, 60)])
def test_lists_that_run_out(settings, item_list, item_points, dtype):
    ctx, n = settings, 5000
    ctx.set_item_list(item_list)
    ctx.set_item_points(item_points)
    Y, csr = embedding(n, "late", dtype), _csr(n, dtype)
    g, z, st = _run(ctx, Y, csr)
    Yo = Y.astype(np.float64)
    go, zo, cnt = oracle.gradient_bh(Yo, csr[0], csr[1], csr[2].astype(np.float64), oracle.Tree(Yo, 20), 0.5, 12.0)
    assert int(st[5]) == n * (n - 1)
    if dtype == np.float64:
        assert st[:3].tolist() == [cnt["tests"], cnt["accepts"], cnt["pairs"]]
    assert rel(g.cpu().numpy(), go) < (1e-10 if dtype == np.float64 else 1e-4)
    assert float(z) == pytest.approx(zo, rel=1e-10 if dtype == np.float64 else 1e-5)


# cells of more than 2048 points are walked whole, by whatever launch
@pytest.mark.parametrize("item_points", [2048, 2049, 1 << 20])
def test_cell_sizes_around_the_largest_walked_in_parts(settings, item_points):
    ctx, sizes = settings, [5000, 700]
    ctx.set_item_points(item_points)
    alone = []
    for j, n in enumerate(sizes):
        Y, csr = embedding(n, "late", np.float32, seed=5 + j), _csr(n, np.float32)
        g, z, st = _run(ctx, Y, csr)
        Yo = Y.astype(np.float64)
        go, zo, _ = oracle.gradient_bh(Yo, csr[0], csr[1], csr[2].astype(np.float64), oracle.Tree(Yo, 20), 0.5, 12.0)
        assert int(st[5]) == n * (n - 1)
        assert rel(g.cpu().numpy(), go) < 1e-4
        assert float(z) == pytest.approx(zo, rel=1e-5)
        alone.append((Y, csr, g, z))
    # the jobs side by side: the same to the bit
    (Y0, c0, g0, z0), (Y1, c1, g1, z1) = alone
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (
        np.concatenate([Y0, Y1]), np.concatenate([c0[0], c1[0][1:] + c0[0][-1]]),
        np.concatenate([c0[1], c1[1] + sizes[0]]).astype(np.int32), np.concatenate([c0[2], c1[2]]))]
    tree = hts.Tree(ctx, sum(sizes), 20)
    tree.set_jobs(sizes)
    hts.build_polar_tree(ctx, dev[0], tree)
    ex = torch.full((2,), 12.0, dtype=torch.float64, device="cuda")
    g, z = hts.gradient_bh_jobs(ctx, *dev, tree, ex, 0.5)
    torch.cuda.synchronize()
    tree.close()
    assert torch.equal(g, torch.cat([g0, g1])) and torch.equal(z, torch.cat([z0, z1]))
