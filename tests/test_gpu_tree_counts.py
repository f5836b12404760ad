"""Counts of a tree of more points than single precision counts one by one (2^24;
depth caps of 1 and 2 admit as many): a node's points are those from its first one
up to the first one of the node after its subtree."""
import numpy as np
import pytest
import torch

from paper_2401_13708_amd import hts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_depth", [1, 2])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_counts_above_two_to_the_24(ctx, max_depth, dtype):
    n = 2 ** 24 + 1
    g = torch.Generator(device="cuda").manual_seed(7)
    Y = (torch.rand(n, 2, generator=g, device="cuda") - 0.5).to(dtype)
    tree = hts.Tree(ctx, n, max_depth)
    hts.build_polar_tree(ctx, Y, tree)
    t = hts.tree_export(ctx, tree, n)
    tree.close()
    assert ctx.check() == 0
    first = np.append(t["first"], n).astype(np.int64)
    assert t["count"][0] == n
    assert np.array_equal(t["count"], first[t["next"]] - first[:-1])
