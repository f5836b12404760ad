"""Rows of P of input points that coincide: the first of them are the neighbours
of all, so several rows longer than a wave sorts follow each other.  Against the
oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2401_13708_amd import hts, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,equal,at", [(513, 513, 0), (1303, 1303, 0), (2000, 700, 0), (2001, 700, 1301)])
def test_equal_points(ctx, n, equal, at):
    k = 30
    X = synth.rng(n).normal(size=(n, 6))
    X[at:at + equal] = X[at]
    knn, rp, col, val = hts.build_affinities(ctx, torch.from_numpy(X).cuda(), 10.0, k)
    oknn, orp, ocol, oval = oracle.build_affinities(X, 10.0, k)
    assert np.array_equal(knn.cpu().numpy(), oknn)
    assert np.array_equal(rp.cpu().numpy(), orp)
    assert np.diff(orp).max() >= equal - 1
    assert np.array_equal(col.cpu().numpy(), ocol)
    # the bandwidths agree to about 1e-9, the entropy's own rounding
    assert np.allclose(val.cpu().numpy(), oval, rtol=1e-7, atol=0)
