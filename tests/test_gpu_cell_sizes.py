"""The upper edges of the rule for the cell size in double precision (64, 128 and 288
points a cell), against the oracle."""
import numpy as np
import pytest

from gpu_inputs import embedding
from test_gpu_walks import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stage", ["init", "late"])
@pytest.mark.parametrize("n", [20479, 20480, 32767, 32768])
def test_sizes_at_the_upper_edges(ctx, n, stage):
    _check(ctx, embedding(n, stage, np.float64))
