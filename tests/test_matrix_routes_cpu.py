"""Which kernels a problem is given, and how much scratch it is told to bring, on the
CPU: the rules are host code that touches no device."""
import pytest

from paper_1905_13298_amd import _native, ops


def test_pixel_counts_near_2_31_keep_off_the_matrix_cores():
    """A tile's pixel range is formed in 32 bits, past its 256 pixels: 8 x 16383 x 16385
    outputs end 8 short of 2^31, where the last tile's end does not fit."""
    n, oh, ow = 8, 16383, 16385
    assert 2 ** 31 - 256 < n * oh * ow < 2 ** 31
    d = ops.describe_conv2d(n, 1, 1, 3, 1, 1, 1, 8191)
    assert "matrix cores" not in d
    # one image fewer is far from the limit
    assert "matrix cores" in ops.describe_conv2d(n - 1, 1, 1, 3, 1, 1, 1, 8191)
