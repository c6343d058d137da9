"""GPU parity of the table form of the small-batch LinearShift (large weights), bit for
bit against the oracle: channels around a 512-thread workgroup and a wave, rows
around the 4 of a table entry, packed rows around the 16 words read at a time and
the words of one table, every code of 2-5 bits, extreme inputs, bias and ReLU."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_13298_amd import ops

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

SHAPES = [
    # batch, in, out, code bits
    (1, 1, 1, 5), (1, 95, 64, 5), (1, 97, 511, 5), (1, 400, 513, 5), (1, 9001, 300, 5), (2, 500, 65, 5),
    (3, 577, 130, 5), (4, 384, 64, 5), (5, 1000, 600, 5), (9, 191, 40, 5), (255, 100, 70, 5),
    (1, 3000, 260, 4), (2, 1000, 70, 3), (4, 777, 100, 2), (7, 129, 33, 3), (1, 20000, 64, 2),
]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"{b}x{c}to{k}b{bits}" for b, c, k, bits in SHAPES])
def test_table_linear_matches_oracle(shape, knob):
    b, c, k, bits = shape
    rng = np.random.default_rng(b * 1000003 + c * 1009 + k)
    x = rng.integers(-(2 ** 31), 2 ** 31, (b, c), dtype=np.int64).astype(np.int32)
    x.flat[:min(x.size, 4)] = [-(2 ** 31), 2 ** 31 - 1, -1, 0][:min(x.size, 4)]
    half = 1 << (bits - 1)
    raw = rng.integers(0, 2 * half, (k, c))
    codes = ((raw // half) << 4 | np.where(raw % half == half - 1, 15, raw % half)).astype(np.uint8)
    bias = rng.integers(-(2 ** 31), 2 ** 31, k, dtype=np.int64).astype(np.int32)
    xt = torch.from_numpy(x).to(DEV)
    wt = torch.from_numpy(ops.pack_shift_weights(codes, bits).view(np.int32)).to(DEV)
    bt = torch.from_numpy(bias).to(DEV)
    knob("DS_ROWS_BATCH", 16)
    print(shape, flush=True)
    y = ops.linear_shift(xt, wt, bt, code_bits=bits).cpu().numpy()
    np.testing.assert_array_equal(y, oracle.linear_shift(x, codes, bias))
    y = ops.linear_shift(xt, wt, None, relu=True, code_bits=bits).cpu().numpy()
    np.testing.assert_array_equal(y, np.maximum(oracle.linear_shift(x, codes, None), 0))
