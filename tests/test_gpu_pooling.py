"""Pooling at the sizes where a window or a plane meets an edge: windows with their
loads unrolled (2 x 2, 3 x 3) and not, padding of half a window, inputs as small as the
window, and planes around the sixteen lanes that sum one. Integers: exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_13298_amd import ops

pytestmark = pytest.mark.gpu


def to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("shape", [(1, 1, 1, 1, 3, 1, 1), (2, 3, 1, 9, 3, 2, 1), (1, 2, 9, 1, 3, 1, 1),
                                   (2, 3, 5, 7, 2, 2, 1), (1, 5, 2, 2, 2, 2, 0), (3, 2, 6, 5, 5, 1, 2),
                                   (1, 2, 11, 8, 4, 3, 2), (2, 7, 33, 31, 3, 2, 0)])
def test_maxpool_edges(shape):
    n, c, h, w, r, st, pd = shape
    x = np.random.default_rng(h * w + r).integers(-(2 ** 31), 2 ** 31 - 1, (n, c, h, w), dtype=np.int64).astype(np.int32)
    x[0, 0] = -(2 ** 31)      # the smallest integer all through a plane
    y = ops.maxpool2d(to_dev(x), r, st, pd).cpu().numpy()
    np.testing.assert_array_equal(y, oracle.maxpool2d(x, r=r, stride=st, pad=pd))


@pytest.mark.parametrize("shape", [(1, 1, 3, 5), (1, 17, 4, 4), (5, 33, 1, 17), (1, 16, 31, 1), (2, 1, 56, 57),
                                   (3, 300, 2, 2), (2, 1000, 1, 1)])
def test_avgpool_edges(shape):
    x = np.random.default_rng(sum(shape)).integers(-(2 ** 31), 2 ** 31 - 1, shape, dtype=np.int64).astype(np.int32)
    x[0, 0] = -(2 ** 31)
    y = ops.avgpool2d_global(to_dev(x)).cpu().numpy()
    np.testing.assert_array_equal(y, oracle.avgpool_global(x))
