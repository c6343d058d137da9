"""GPU parity of the matrix-core kernels, bit for bit against the oracle: the edges
of their tiles (256 pixels, 64 channels, 32-channel blocks, chunks of two blocks,
odd block counts, tap columns folded into channels), inputs inside the one-digit
range, at its edges, beyond it in some blocks only and over all of int32, sums
that reach the exact range of the accumulators, split reductions, both output
layouts, the fused epilogue and 2-5-bit codes. Variant 64 forces the kernels
where the problem is too small for them to be the automatic choice."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_13298_amd import ops
from paper_1905_13298_amd.workloads import random_codes

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def to_dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def inputs(rng, mode, shape):
    if mode == "digit":       # |x| < 2^20: one digit above the low 16 bits
        x = rng.integers(-(2 ** 20), 2 ** 20, shape)
    elif mode == "edges":     # either side of that range, and the type's ends
        x = rng.choice([-(2 ** 31), 2 ** 31 - 1, -(2 ** 20) - 1, -(2 ** 20), 2 ** 20 - 1, 2 ** 20, -1, 0, 1], shape)
    elif mode == "one":       # a single value beyond it
        x = rng.integers(0, 2 ** 18, shape)
        x[-1, -1, -1, -1] = -(2 ** 31)
    elif mode == "spots":     # a few, in some tiles' windows only
        x = rng.integers(0, 2 ** 18, shape)
        spots = rng.choice(x.size, 6, replace=False)
        x.flat[spots] = rng.integers(-(2 ** 31), 2 ** 31, 6)
    elif mode in ("two", "three", "four"):   # what is above bit 15 at the ends of two or three digits, or past them
        ends = {"two": [-528, -17, 16, 495], "three": [-16912, -529, 496, 15855], "four": [-32768, -16913, 15856, 32767]}
        x = rng.choice(ends[mode] + [0], shape) * 65536 + rng.integers(0, 65536, shape)
    elif mode == "mixed":     # values of one to four digits, few enough that some tiles and blocks have none
        x = rng.integers(0, 2 ** 18, shape)
        spots = rng.choice(x.size, 8, replace=False)
        x.flat[spots] = rng.choice([-1, 1], 8) * 2 ** np.array([19, 21, 24, 26, 29, 30, 22, 27])
    else:                     # "full": all of int32
        x = rng.integers(-(2 ** 31), 2 ** 31, shape, dtype=np.int64)
    return x.astype(np.int32)


CASES = [
    # n, c, h, w, k, r, s, stride, pad, inputs
    (1, 1, 1, 257, 1, 1, 1, 1, 0, "full"),        # one channel, one pixel past a tile
    (1, 32, 16, 16, 64, 1, 1, 1, 0, "digit"),     # exactly one tile, one block
    (1, 64, 16, 16, 65, 1, 1, 1, 0, "edges"),     # one channel past a row tile
    (3, 40, 9, 9, 65, 1, 1, 2, 0, "one"),         # strided 1 x 1: a packed copy of the sampled pixels
    (2, 96, 14, 14, 70, 3, 3, 2, 1, "edges"),     # odd number of blocks: a chunk spans two taps
    (2, 33, 13, 17, 70, 3, 2, 2, 1, "full"),      # ragged channels, window and rows
    (1, 3, 40, 41, 64, 7, 7, 2, 3, "digit"),      # folded tap columns
    (2, 10, 11, 12, 33, 5, 3, 1, 2, "full"),      # folded, padding beyond the window's half
    (2, 64, 7, 7, 128, 3, 3, 1, 1, "digit"),      # small images: a tile spans several
    (300, 256, 1, 1, 128, 1, 1, 1, 0, "digit"),   # LinearShift: y in rows of channels
    (261, 250, 1, 1, 130, 1, 1, 1, 0, "full"),    # unaligned rows
    # images of many tiles: values beyond one digit reach the tiles whose rows hold them
    (1, 32, 70, 90, 64, 3, 3, 1, 1, "spots"),
    (2, 40, 61, 50, 64, 5, 3, 2, 2, "spots"),
    (1, 3, 90, 83, 64, 7, 7, 2, 3, "spots"),      # folded
    (3, 33, 35, 41, 64, 1, 1, 2, 0, "spots"),     # sampled
    (1, 32, 50, 60, 64, 3, 3, 1, 9, "spots"),     # tiles whose rows lie in the padding
    (1, 32, 40, 300, 64, 3, 1, 3, 0, "one"),      # rows wider than a tile
    # every number of digits, whole and split, odd and even block counts, past a tile's edges
    (2, 40, 13, 21, 70, 3, 3, 1, 1, "two"),
    (2, 72, 13, 21, 70, 3, 3, 1, 1, "three"),
    (2, 40, 13, 21, 70, 1, 1, 1, 0, "three"),
    (2, 64, 13, 21, 70, 3, 3, 1, 1, "four"),
    (1, 96, 60, 50, 65, 3, 3, 1, 1, "mixed"),
    (2, 3, 61, 50, 64, 7, 7, 2, 3, "mixed"),      # folded
    (300, 130, 1, 1, 130, 1, 1, 1, 0, "mixed"),
]


@pytest.mark.parametrize("case", CASES, ids=[f"{i}_{c[-1]}" for i, c in enumerate(CASES)])
def test_matrix_core_convolutions_match_oracle(case, knob):
    n, c, h, w, k, r, s, stride, pad, mode = case
    rng = np.random.default_rng(100 + CASES.index(case))
    x = inputs(rng, mode, (n, c, h, w))
    codes = random_codes(rng, (k, c * r * s), zero_frac=0.1)
    bias = rng.integers(-(2 ** 31), 2 ** 31, k, dtype=np.int64).astype(np.int32)
    knob("DS_FORCE_VARIANT", 64)
    assert ops.describe_conv2d(n, c, h, w, k, (r, s), stride, pad).startswith("matrix cores")
    print(case, ops.describe_conv2d(n, c, h, w, k, (r, s), stride, pad), flush=True)
    want = oracle.conv2d_shift(x, codes, bias, r=r, s=s, stride=stride, pad=pad)
    size = want.size
    big = torch.full((size + 512,), 0x5A5A5A5A, dtype=torch.int32, device=DEV)   # canaries around y
    y = ops.conv2d_shift(to_dev(x), to_dev(ops.pack_shift_weights(codes).view(np.int32)), to_dev(bias), (r, s),
                         stride, pad, out=big[256:256 + size].view(want.shape))
    np.testing.assert_array_equal(y.cpu().numpy(), want)
    edge = big.cpu().numpy()
    assert np.all(edge[:256] == 0x5A5A5A5A) and np.all(edge[256 + size:] == 0x5A5A5A5A)


@pytest.mark.parametrize("value,shift", [(2 ** 20 - 1, 6), (-(2 ** 20), 6), (2 ** 20 - 1, 0), (2 ** 31 - 1, 0),
                                         (15855 * 2 ** 16 + 65535, 6), (-16912 * 2 ** 16, 0), (-(2 ** 31), 6)])
def test_sums_past_the_accumulators_exact_range(value, shift, knob):
    """1056 equal terms of the largest size an accumulator meets (shift 6 in one, shift
    0 in the other): a tile that walked them in one go would pass 2^24 units. The grid
    is large enough that the reduction is not split."""
    n, c, k = 300, 1056, 16
    knob("DS_FORCE_VARIANT", 64)
    assert ops.describe_conv2d(n, c, 16, 16, k, 1).startswith("matrix cores, parts 1;")
    x = torch.full((n, c, 16, 16), value, dtype=torch.int32, device=DEV)
    codes = np.full((k, c), shift, dtype=np.uint8)
    codes[1::2] |= 16
    y = ops.conv2d_shift(x, to_dev(ops.pack_shift_weights(codes).view(np.int32)), None, 1)
    total = c * (value >> shift)
    wrap = lambda v: (v + 2 ** 31) % 2 ** 32 - 2 ** 31
    assert torch.all(y[:, 0::2] == wrap(total)) and torch.all(y[:, 1::2] == wrap(-total))


@pytest.mark.parametrize("mode", ["digit", "edges"])
@pytest.mark.parametrize("shape", [(96, 64, 16, 64, 1), (2, 128, 14, 100, 3), (260, 64, 1, 72, 1), (3, 40, 9, 65, 1)],
                         ids=["whole", "split", "linear", "ragged"])
def test_matrix_core_epilogue_matches_oracle(shape, mode, knob):
    n, c, h, k, r = shape
    rng = np.random.default_rng(n + c)
    x = inputs(rng, mode, (n, c, h, h))
    codes = random_codes(rng, (k, c * r * r), zero_frac=0.1)
    bias, mul, add = (rng.integers(-(2 ** 18), 2 ** 18, k).astype(np.int32) for _ in range(3))
    res = rng.integers(-(2 ** 31), 2 ** 31, (n, k, h, h), dtype=np.int64).astype(np.int32)
    knob("DS_FORCE_VARIANT", 64)
    # ragged: one launch applies the epilogue to a last wave of 51 pixels and to one
    # channel past a row tile, each lane's parameters being another channel's
    if shape == (3, 40, 9, 65, 1):
        assert ops.describe_conv2d(n, c, h, h, k, r, 1, r // 2).startswith("matrix cores, parts 1;")
    y = ops.conv2d_shift_fused(to_dev(x), to_dev(ops.pack_shift_weights(codes).view(np.int32)), to_dev(bias), r, 1,
                               r // 2, mul=to_dev(mul), add=to_dev(add), mul_shift=13, residual=to_dev(res), relu=True)
    want = oracle.epilogue(oracle.conv2d_shift(x, codes, bias, r=r, stride=1, pad=r // 2), mul, add, 13, res, True)
    np.testing.assert_array_equal(y.cpu().numpy(), want)


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_matrix_core_short_codes_match_oracle(bits, knob):
    rng = np.random.default_rng(bits)
    x = inputs(rng, "digit", (2, 64, 9, 9))
    codes = random_codes(rng, (70, 64 * 9), zero_frac=0.2, max_shift=(1 << (bits - 1)) - 2)
    knob("DS_FORCE_VARIANT", 64)
    y = ops.conv2d_shift(to_dev(x), to_dev(ops.pack_shift_weights(codes, bits).view(np.int32)), None, 3, 1, 1,
                         code_bits=bits)
    np.testing.assert_array_equal(y.cpu().numpy(), oracle.conv2d_shift(x, codes, None, r=3, stride=1, pad=1))


GRADS = [
    # n, c, h, w, k, r, s, stride, pad
    (2, 64, 14, 14, 32, 3, 3, 1, 1),      # one phase, dense
    (2, 70, 16, 16, 33, 3, 3, 2, 1),      # four phases on one packed copy, ragged channels
    (2, 40, 15, 13, 64, 3, 3, 2, 0),      # phase grids of different sizes
    (1, 20, 20, 21, 40, 7, 7, 2, 3),      # four phases of 3 and 4 taps
    (2, 33, 12, 12, 40, 1, 1, 2, 0),      # positions no tap reaches
    (2, 20, 14, 14, 24, 5, 5, 3, 2),      # nine phases: groups of four tasks
    (1, 17, 9, 9, 24, 3, 3, 1, 4),        # padding beyond the window
    (260, 100, 1, 1, 130, 1, 1, 1, 0),    # LinearShift
]


@pytest.mark.parametrize("mode", ["digit", "edges"])
@pytest.mark.parametrize("case", GRADS, ids=[str(i) for i in range(len(GRADS))])
def test_matrix_core_gradients_match_oracle(case, mode, knob):
    """Calls and plans, every element of dx written."""
    n, c, h, w, k, r, s, stride, pad = case
    rng = np.random.default_rng(GRADS.index(case))
    oh, ow = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - s) // stride + 1
    dy = inputs(rng, mode, (n, k, oh, ow))
    codes = random_codes(rng, (k, c * r * s), zero_frac=0.1)
    knob("DS_FORCE_VARIANT", 64)
    assert ops.describe_conv2d_backward_data(n, c, h, w, k, (r, s), stride, pad).startswith("matrix cores; else ")
    print(case, mode, flush=True)
    want = oracle.conv2d_shift_backward_data(dy, codes, (n, c, h, w), r=r, s=s, stride=stride, pad=pad)
    wp = ops.pack_shift_weights(codes)
    out = torch.full((n, c, h, w), 0x5A5A5A5A, dtype=torch.int32, device=DEV)
    dx = ops.conv2d_shift_backward_data(to_dev(dy), to_dev(wp.view(np.int32)), (n, c, h, w), (r, s), stride, pad, out=out)
    np.testing.assert_array_equal(dx.cpu().numpy(), want)
    plan = ops.JitConvBackwardData(wp, (n, c, h, w), (r, s), stride, pad)
    assert plan.matrix_cores
    out.fill_(0x5A5A5A5A)
    np.testing.assert_array_equal(plan(to_dev(dy), out=out).cpu().numpy(), want)
    plan.close()


@pytest.mark.parametrize("act_bits", [32, 16, 8])
@pytest.mark.parametrize("shape", [(96, 64, 16, 64, 1, 1, 0), (2, 100, 14, 100, 3, 1, 1), (2, 3, 30, 40, 7, 2, 3),
                                   (260, 64, 1, 72, 1, 1, 0), (3, 40, 18, 65, 1, 2, 0)],
                         ids=["whole", "split", "folded", "linear", "ragged"])
def test_matrix_core_plans_match_oracle(shape, act_bits, knob):
    """Plans of every input width with the whole epilogue, run twice on new inputs, the
    second time as replays of a captured graph."""
    n, c, h, k, r, stride, pad = shape
    rng = np.random.default_rng(n + c + act_bits)
    codes = random_codes(rng, (k, c * r * r), zero_frac=0.1)
    bias, mul, add = (rng.integers(-(2 ** 18), 2 ** 18, k).astype(np.int32) for _ in range(3))
    knob("DS_FORCE_VARIANT", 64)
    plan = ops.JitConv(ops.pack_shift_weights(codes), (n, c, h, h), r, stride, pad, bias=bias, mul=mul, add=add,
                       mul_shift=13, residual=True, relu=True, act_bits=act_bits)
    assert plan.matrix_cores and plan.preferred
    dtype = {32: np.int32, 16: np.int16, 8: np.int8}[act_bits]

    def draw():
        info = np.iinfo(dtype)
        x = rng.integers(info.min, info.max + 1, (n, c, h, h), dtype=np.int64).astype(dtype)
        res = rng.integers(-(2 ** 31), 2 ** 31, plan.y_shape, dtype=np.int64).astype(np.int32)
        v = oracle.conv2d_shift(x.astype(np.int32), codes, bias, r=r, stride=stride, pad=pad)
        return x, res, oracle.epilogue(v, mul, add, 13, res, True)

    x, res, want = draw()
    xt, rt = to_dev(x), to_dev(res)
    y = plan(xt, residual=rt)
    np.testing.assert_array_equal(y.cpu().numpy(), want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan(xt, residual=rt, out=y)
    for _ in range(3):
        x, res, want = draw()
        xt.copy_(to_dev(x))
        rt.copy_(to_dev(res))
        y.fill_(7)
        graph.replay()
        np.testing.assert_array_equal(y.cpu().numpy(), want)
    plan.close()


def test_scratch_entry_points(knob):
    """Scratch given to a call, too little of it (the call then allocates), none, and
    bad scratch, which is refused before anything runs."""
    import ctypes
    from paper_1905_13298_amd import _native
    lib = _native.lib()
    rng = np.random.default_rng(5)
    n, c, h, k = 2, 40, 12, 70
    x = inputs(rng, "digit", (n, c, h, h))
    codes = random_codes(rng, (k, c * 9))
    want = oracle.conv2d_shift(x, codes, None, r=3, stride=1, pad=1)
    xt, wt = to_dev(x), to_dev(ops.pack_shift_weights(codes).view(np.int32))
    shape = (n, c, h, h, k, 3, 3, 1, 1, 1, 1)
    stream = ctypes.c_void_p(torch.cuda.current_stream(DEV).cuda_stream)
    for variant in (64, 4):
        knob("DS_FORCE_VARIANT", variant)
        need = lib.ds_conv2d_shift_scratch_bytes(*shape)
        buf = torch.empty(need + 256, dtype=torch.uint8, device=DEV)
        for ptr, size, status in ((buf.data_ptr(), need, 0), (buf.data_ptr(), need - 1, 0), (None, 0, 0),
                                  (buf.data_ptr() + 4, need, 3), (buf.data_ptr(), 1 << 40, 3), (xt.data_ptr(), 256, 3)):
            y = torch.full(want.shape, 7, dtype=torch.int32, device=DEV)
            st = lib.ds_conv2d_shift_fused_ws(xt.data_ptr(), wt.data_ptr(), None, None, None, 0, None, y.data_ptr(),
                                              *shape, 16, 0, ptr, size, stream)
            assert st == status, (variant, size, st)
            if status == 0:
                np.testing.assert_array_equal(y.cpu().numpy(), want)
            else:
                assert torch.all(y == 7)


@pytest.mark.parametrize("variant", [64, 4])
def test_scratch_over_any_buffer_is_refused(variant, knob):
    """Scratch that shares memory with any of a call's buffers, by one word at either end,
    is refused and nothing is written; next to them it is taken."""
    import ctypes
    from paper_1905_13298_amd import _native
    lib = _native.lib()
    rng = np.random.default_rng(6)
    n, c, h, k = 2, 40, 12, 70
    x = inputs(rng, "digit", (n, c, h, h))
    codes = random_codes(rng, (k, c * 9))
    bias, mul, add = (rng.integers(-(2 ** 18), 2 ** 18, k).astype(np.int32) for _ in range(3))
    res = rng.integers(-(2 ** 20), 2 ** 20, (n, k, h, h)).astype(np.int32)
    knob("DS_FORCE_VARIANT", variant)
    shape = (n, c, h, h, k, 3, 3, 1, 1, 1, 1)
    need = max(lib.ds_conv2d_shift_scratch_bytes(*shape), lib.ds_conv2d_shift_backward_data_scratch_bytes(*shape))
    need = (need + 255) // 256 * 256
    data = dict(x=x, w=ops.pack_shift_weights(codes).view(np.int32), bias=bias, mul=mul, add=add, res=res, y=res)
    stream = ctypes.c_void_p(torch.cuda.current_stream(DEV).cuda_stream)
    # every buffer between two stretches of scratch, all starting on 256-byte boundaries
    room, at = {}, need
    for name, a in data.items():
        room[name] = at
        at += (a.nbytes + 255) // 256 * 256 + need
    big = torch.zeros(at, dtype=torch.uint8, device=DEV)
    base = big.data_ptr()
    view = {m: big[room[m]:room[m] + a.nbytes].view(torch.int32).view(a.shape) for m, a in data.items()}
    for m, a in data.items():
        view[m].copy_(torch.from_numpy(a))
    view["y"].fill_(7)
    p = {m: base + room[m] for m in data}

    def forward(scratch):
        return lib.ds_conv2d_shift_fused_ws(p["x"], p["w"], p["bias"], p["mul"], p["add"], 13, p["res"], p["y"], *shape,
                                            16, 1, scratch, need, stream)

    def gradient(scratch):
        return lib.ds_conv2d_shift_backward_data_ws(p["res"], p["w"], p["x"], *shape, 16, 0, scratch, need, stream)

    before = big.clone()
    for m, a in data.items():
        ends = [p[m] - need + 256, p[m] + (a.nbytes - 1) // 256 * 256]
        for scratch in ends:
            assert forward(scratch) == 3, m
            if m in ("res", "w", "x"):
                assert gradient(scratch) == 3, m
    assert torch.equal(big, before)
    assert forward(p["w"] - need) == 0
    v = oracle.conv2d_shift(x, codes, bias, r=3, stride=1, pad=1)
    np.testing.assert_array_equal(view["y"].cpu().numpy(), oracle.epilogue(v, mul, add, 13, res, True))
    assert gradient(p["y"] - need) == 0
    want = oracle.conv2d_shift_backward_data(res, codes, (n, c, h, h), r=3, stride=1, pad=1)
    np.testing.assert_array_equal(view["x"].cpu().numpy(), want)
