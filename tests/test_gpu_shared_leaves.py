"""Trees whose leaves hold several points (depth caps, equal points): their cells are
handed over whole up to the default size, and walked whole beside chunks in parts; the
oracle's gradient, the same bits in every launch shape and alone or in a layout."""
import numpy as np
import pytest
import torch

from paper_2401_13708_amd import hts, synth
from gpu_inputs import embedding, rel
from test_gpu_parts import _both, _check as check_f32, _csr
from test_gpu_walks import _check as check_f64

pytestmark = pytest.mark.gpu

# points, depth cap, copies of each point: whole chunks only, both kinds, nodes and
# points about equal, leaves of more than a cell and of more than 288 points, every
# launch rule
CASES = [(300, 2, 1), (1000, 4, 1), (1000, 8, 1), (3000, 10, 1), (3000, 20, 16), (3000, 20, 128), (3100, 20, 300),
         (6100, 20, 64), (9000, 8, 1), (12287, 20, 250), (12288, 20, 64)]


def _points(n, copies, dtype):
    base = embedding(max(2, n // copies), "late", dtype)
    return np.ascontiguousarray(base[np.arange(n) % base.shape[0]])


@pytest.mark.parametrize("theta", [0.0, 0.5])
@pytest.mark.parametrize("n,depth,copies", CASES)
def test_single(ctx, n, depth, copies, theta):
    check_f32(ctx, _points(n, copies, np.float32), max_depth=depth, theta=theta)


@pytest.mark.parametrize("n,depth,copies", CASES + [(20479, 20, 250)])
def test_double(ctx, n, depth, copies):
    check_f64(ctx, _points(n, copies, np.float64), theta=0.0, max_depth=depth)


@pytest.mark.parametrize("item_list", [hts.DEFAULT_ITEM_LIST, 3])
@pytest.mark.parametrize("n,depth,copies", CASES + [(20479, 20, 250)])
def test_double_as_with_small_cells_only(ctx, n, depth, copies, item_list):
    # the same terms in another order: a few hundred units of 2^-53 of the largest.
    # (Midpoints of equal points near the rim are the oracle's to 1e-9 only: both round
    # a sum whose distance to the rim counts.)
    Y = _points(n, copies, np.float64)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
           for a in (Y, *synth.random_csr(n, min(20, n // 4), seed=3, dtype=np.float64))]
    tree = hts.Tree(ctx, n, depth)
    hts.build_polar_tree(ctx, dev[0], tree)
    try:
        ctx.set_item_list(item_list)
        g, z = hts.gradient_bh(ctx, *dev, tree, 0.5, 12.0)
        ctx.set_item_points(32)
        g2, z2 = hts.gradient_bh(ctx, *dev, tree, 0.5, 12.0)
        torch.cuda.synchronize()
        assert ctx.check() == 0
    finally:
        ctx.set_item_points(hts.DEFAULT_ITEM_POINTS)
        ctx.set_item_list(hts.DEFAULT_ITEM_LIST)
    tree.close()
    assert rel(g.cpu().numpy(), g2.cpu().numpy()) < 1e-12
    assert float(z) == pytest.approx(float(z2), rel=1e-12)


@pytest.mark.parametrize("n,copies", [(3000, 128), (3000, 250), (10000, 200)])
def test_cells_that_cannot_be_divided_are_handed_over(ctx, n, copies):
    # in double precision cells are of 64 points at these sizes; a leaf that holds more
    # is the second phase's all the same (walked by the first: 163 and 300 us, n = 3000)
    Y = _points(n, copies, np.float64)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
           for a in (Y, *synth.random_csr(n, 20, seed=3, dtype=np.float64))]
    tree = hts.Tree(ctx, n, 20)
    hts.build_polar_tree(ctx, dev[0], tree)
    st = torch.zeros(hts.STATS_PER_CALL, dtype=torch.int64, device="cuda")
    hts.gradient_bh(ctx, *dev, tree, 0.0, 1.0, stats=st)
    torch.cuda.synchronize()
    tree.close()
    st = st.tolist()
    assert st[2] == n * (n - 1)
    assert st[6 + 2] >= 0.9 * st[2]


@pytest.mark.parametrize("n,depth,copies", [(1000, 4, 1), (3000, 20, 64), (6100, 20, 64), (9000, 8, 1)])
def test_hsne(ctx, n, depth, copies):
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (_points(n, copies, np.float32), *_csr(n))]
    tree = hts.Tree(ctx, n, depth)
    hts.build_polar_tree(ctx, dev[0], tree)

    def run():
        g, z = hts.gradient_hsne(ctx, *dev, tree, lam=0.8, theta=0.2)
        torch.cuda.synchronize()
        return g, z

    _both(ctx, run)
    tree.close()


def test_jobs_alone_and_beside_others(ctx):
    sizes, copies = [3000, 500, 13000, 2000, 64], [64, 1, 100, 16, 32]
    n = sum(sizes)
    Ys = [_points(m, c, np.float32) for m, c in zip(sizes, copies)]
    csr = [_csr(m) for m in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)])
    nnz = np.concatenate([[0], np.cumsum([c[0][-1] for c in csr])])
    rp = np.concatenate([[0]] + [c[0][1:] + nnz[j] for j, c in enumerate(csr)]).astype(np.int64)
    col = np.concatenate([c[1] + off[j] for j, c in enumerate(csr)]).astype(np.int32)
    val = np.concatenate([c[2] for c in csr]).astype(np.float32)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (np.concatenate(Ys), rp, col, val)]
    tree = hts.Tree(ctx, n, 20)
    tree.set_jobs(sizes)
    hts.build_polar_tree(ctx, dev[0], tree)
    ex = torch.ones(len(sizes), dtype=torch.float64, device="cuda")
    g, z = hts.gradient_bh_jobs(ctx, *dev, tree, ex, 0.2)
    torch.cuda.synchronize()
    tree.close()
    for j, m in enumerate(sizes):
        one = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (Ys[j], *csr[j])]
        t = hts.Tree(ctx, m, 20)
        hts.build_polar_tree(ctx, one[0], t)
        gs, zs = hts.gradient_bh(ctx, *one, t, 0.2, 1.0)
        torch.cuda.synchronize()
        t.close()
        assert torch.equal(g[off[j]:off[j + 1]], gs), j
        assert float(z[j]) == float(zs[0]), j
    assert ctx.check() == 0
