"""h-SNE in single precision against the oracle at the edges of its launch rules: the
waves of a workgroup share a chunk below 6144 points over both metrics (8 waves), below
12288 (4), none from there on. The bar is that of every single-precision h-SNE gradient."""
import numpy as np
import pytest
import torch

import oracle
from paper_2401_13708_amd import hts, synth
from gpu_inputs import embedding, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stage", ["init", "late"])
@pytest.mark.parametrize("n", [100, 3071, 3072, 6143, 6144])
def test_both_traversals_match_the_oracle(ctx, n, stage):
    Y = embedding(n, stage, np.float32)
    rp, col, val = synth.random_csr(n, min(20, max(1, n // 4)), seed=3, dtype=np.float32)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (Y, rp, col, val)]
    tree = hts.Tree(ctx, n, 20)
    hts.build_polar_tree(ctx, dev[0], tree)
    g, z = hts.gradient_hsne(ctx, *dev, tree, lam=0.8, theta=0.5, exaggeration=12.0)
    torch.cuda.synchronize()
    assert ctx.check() == 0
    tree.close()
    Yo, vo = Y.astype(np.float64), val.astype(np.float64)
    t = oracle.Tree(Yo, 20)
    ge, ze, _ = oracle.gradient_euclid_bh(Yo, rp, col, vo, t, 0.5, 12.0)
    gh, zh, _ = oracle.gradient_bh(Yo, rp, col, vo, t, 0.5, 12.0)
    assert rel(g.cpu().numpy(), ge + 0.8 * gh) < 1e-3
    assert z.cpu().numpy() == pytest.approx([ze, zh], rel=1e-5)
