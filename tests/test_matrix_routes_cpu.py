"""Which kernels a problem is given, and how much scratch it is told to bring, on the
CPU: the rules are host code that touches no device."""
import pytest

from paper_1905_13298_amd import _native, ops

from .mock_hip import run


def test_pixel_counts_near_2_31_keep_off_the_matrix_cores(knob):
    """A tile's pixel range is formed in 32 bits, past its 256 pixels: 8 x 16383 x 16385
    outputs end 8 short of 2^31, where the last tile's end does not fit."""
    n, oh, ow = 8, 16383, 16385
    knob("DS_FORCE_VARIANT", 64)
    assert 2 ** 31 - 256 < n * oh * ow < 2 ** 31
    d = ops.describe_conv2d(n, 1, 1, 3, 1, 1, 1, 8191)
    assert "matrix cores" not in d
    # one image fewer is far from the limit
    assert "matrix cores" in ops.describe_conv2d(n - 1, 1, 1, 3, 1, 1, 1, 8191)


@pytest.mark.parametrize("shape", [(2, 64, 14, 14, 32, 3, 1, 1), (2, 70, 16, 16, 33, 3, 2, 1), (3, 20, 15, 15, 33, 1, 2, 0)])
def test_gradient_scratch_covers_its_convolutions(shape, knob):
    """On the vector kernels a gradient runs one convolution per stride phase; the scratch
    that the caller is told to bring holds the phase's codes and all that the
    convolution takes (which the call would otherwise allocate)."""
    n, c, h, w, k, r, stride, pad = shape
    lib = _native.lib()
    knob("DS_FORCE_VARIANT", 4)
    oh = (h + 2 * pad - r) // stride + 1
    # the phase of the most taps, as a forward problem on dy (padding does not change its scratch's weights)
    taps = -(-r // stride)
    need = lib.ds_conv2d_shift_scratch_bytes(n, k, oh, oh, c, taps, taps, 1, 1, taps - 1, taps - 1)
    assert need > 0
    assert lib.ds_conv2d_shift_backward_data_scratch_bytes(n, c, h, w, k, r, r, stride, stride, pad, pad) >= need


def test_noalloc_reports_the_scratch_it_uses():
    """A shape that is told to need none stays off the one array; one that the matrix cores
    run there uses their scratch; one whose scratch there would not fit, the vector
    kernels'."""
    lib = _native.lib()
    need = lambda *a: lib.ds_conv2d_shift_noalloc_scratch_bytes(*a)
    matrix = lambda *a: lib.ds_conv2d_shift_scratch_bytes(*a)
    fits = (4, 64, 28, 28, 128, 3, 3, 1, 1, 1, 1)
    assert "matrix cores" in ops.describe_conv2d(4, 64, 28, 28, 128, 3, 1, 1)
    assert need(*fits) == matrix(*fits) < 32 << 20
    none = (1, 64, 56, 56, 64, 6, 6, 1, 1, 2, 2)      # no tiled instance
    assert need(*none) == 0 < matrix(*none)
    large = (64, 64, 112, 112, 64, 3, 3, 1, 1, 1, 1)
    assert 0 < need(*large) < 32 << 20 < matrix(*large)
    assert need(8, 256, 1, 1, 128, 1, 1, 1, 1, 0, 0) == 0


def test_calls_and_plans_without_room_for_the_matrix_cores_run_without_them(tmp_path):
    """Packed inputs and expanded weights take far more memory than what they replace: where
    they cannot be allocated, calls run on the vector kernels and plans on generated
    code, as they did with that little memory before. (Against a stand-in runtime whose
    allocations fail past a limit.)"""
    run("""
wp = np.zeros((256, (256 * 9 + 5) // 6), np.uint32)
buf = np.zeros(1 << 16, np.uint8).ctypes.data
shape = (32, 256, 14, 14, 256, 3, 3, 1, 1, 1, 1)
need = lib.ds_conv2d_shift_scratch_bytes(*shape)
far = [buf + (i << 36) for i in range(4)]         # never touched: launches run nothing
call = lambda: lib.ds_conv2d_shift(far[0], far[1], None, far[2], *shape, 16, 0, None)
grad = lambda: lib.ds_conv2d_shift_backward_data(far[0], far[1], far[2], *shape, 16, 0, None)
for f in (call, grad):
    mock.mock_reset(ALL)
    assert f() == 0 and "mfma_conv_kernel" in kernels(), kernels()
    matrix = mock.mock_largest()
    mock.mock_reset(matrix - 1)
    assert f() == 0, lib.ds_last_error_message()
    assert "tiled_kernel" in kernels() and "mfma_conv_kernel" not in kernels(), kernels()
    assert mock.mock_failures() == 1
    mock.mock_reset(1)                            # nothing can be allocated: an error, as before
    assert f() == 6 and kernels() == []
for create in (lambda p: lib.ds_jit_conv_create(wp.ctypes.data, None, None, None, 0, *shape, 0, 0, p),
               lambda p: lib.ds_jit_conv_backward_data_create(wp.ctypes.data, *shape, 0, 0, p)):
    mock.mock_reset(ALL)
    p = ctypes.c_void_p()
    assert create(ctypes.byref(p)) == 0 and lib.ds_jit_conv_matrix_cores(p) == 1
    matrix = mock.mock_largest()
    lib.ds_jit_conv_destroy(p)
    mock.mock_reset(matrix - 1)
    assert create(ctypes.byref(p)) == 0, lib.ds_last_error_message()
    assert lib.ds_jit_conv_matrix_cores(p) == 0 and "module" in kernels()
    assert lib.ds_jit_conv_run(p, far[0], None, far[2], None) == 0 and "generated" in kernels()
    lib.ds_jit_conv_destroy(p)
""", tmp_path)


def test_plans_of_sparse_weights_are_generated_code(tmp_path):
    """Generated code has an instruction a non-zero weight, the matrix cores' time does not
    depend on them: plans of the same layer take the one or the other by the share of
    zero codes, of any width and with a last word that is not full. (Against a stand-in
    runtime.)"""
    run("""
from paper_1905_13298_amd import ops
shape = (128, 256, 14, 14, 256, 3, 3, 1, 1, 1, 1)
def plan(codes, bits, gradient):
    wp = ops.pack_shift_weights(codes, bits=bits)
    p = ctypes.c_void_p()
    flags = 0 if bits == 5 else ops.code_bits_flag(bits)
    if gradient:
        st = lib.ds_jit_conv_backward_data_create(wp.ctypes.data, *shape, flags, 0, ctypes.byref(p))
    else:
        st = lib.ds_jit_conv_create(wp.ctypes.data, None, None, None, 0, *shape, flags, 0, ctypes.byref(p))
    assert st == 0, lib.ds_last_error_message()
    matrix = lib.ds_jit_conv_matrix_cores(p)
    lib.ds_jit_conv_destroy(p)
    return matrix
mock.mock_reset(ALL)
rng = np.random.default_rng(0)
for bits in (5, 4, 3, 2):
    top = (1 << (bits - 1)) - 1                # its shifts are 0 .. top - 1
    for zeros, matrix in ((0.0, 1), (0.2, 1), (0.5, 1), (0.9, 0), (1.0, 0)):
        sign, shift = rng.integers(0, 2, (256, 2304)), rng.integers(0, top, (256, 2304))
        shift[rng.random(shift.shape) < zeros] = 15
        codes = (sign << 4 | shift).astype(np.uint8)
        for gradient in (False, True):
            assert plan(codes, bits, gradient) == matrix, (bits, zeros, gradient)
""", tmp_path)


def test_small_batch_linear_takes_the_faster_kernel(tmp_path):
    """The choice between the table and the kernel that decodes each code, where they are
    furthest apart (measured on MI355X, us: decoding, table): by codes' width, by long rows
    of few channels and by terms."""
    run("""
x, w, y = (np.zeros(64, np.int32).ctypes.data + (i << 36) for i in range(3))   # never touched
def table(n, c, k, bits):
    mock.mock_reset(ALL)
    flags = 0 if bits == 5 else bits << 8
    assert lib.ds_linear_shift(x, w, None, y, n, c, k, 16, flags, None) == 0, lib.ds_last_error_message()
    names = kernels()
    assert ("linear_table_kernel" in names) != ("linear_rows_kernel" in names), names
    return "linear_table_kernel" in names
for n, c, k, bits in [(1, 25088, 4096, 5), (1, 25088, 512, 5),      # 39.0, 24.5; 17.3, 11.6
                      (128, 4096, 4096, 5), (200, 2048, 2048, 5),   # 233, 157; 121, 78
                      (64, 2048, 1000, 5), (200, 2048, 256, 5),     # 19.5, 14.9; 21.3, 16.2
                      (4, 8000, 256, 2), (1, 8000, 1000, 3), (128, 512, 4096, 4)]:   # 14.1, 8.9; 8.9, 7.1; 37.3, 18.7
    assert table(n, c, k, bits), (n, c, k, bits)
for n, c, k, bits in [(96, 25088, 256, 5), (200, 25088, 256, 5),    # 95.6, 113; 181, 227
                      (32, 512, 1000, 5), (8, 256, 128, 2),         # 5.8, 9.1; fewer than 256 channels
                      (16, 1024, 512, 5), (4, 2048, 1000, 4), (64, 512, 256, 2)]:    # 6.9, 9.2; 6.9, 9.1; 5.4, 9.1
    assert not table(n, c, k, bits), (n, c, k, bits)
""", tmp_path)


def test_short_reductions_keep_off_the_matrix_cores():
    """A chunk is 64 terms: a reduction of a few, most of it padding, runs on the vector kernels
    where it is measured faster there (the comment's figures, us: vector, matrix cores)."""
    matrix = lambda n, c, h, k, r, p: ops.describe_conv2d(n, c, h, h, k, r, 1, p).startswith("matrix cores")
    for shape in [(8, 4, 112, 24, 1, 0), (64, 8, 56, 64, 1, 0), (64, 1, 56, 64, 3, 1), (64, 3, 56, 24, 3, 1)]:
        assert not matrix(*shape), shape        # 14, 20; 26, 39; 29, 45; 34, 44
    for shape in [(2, 3, 512, 64, 3, 1), (64, 16, 56, 128, 1, 0), (8, 24, 112, 64, 1, 0), (64, 64, 28, 64, 1, 0)]:
        assert matrix(*shape), shape            # 104, 75; 55, 49
    grad = lambda n, c, h, k, r, s, p: ops.describe_conv2d_backward_data(n, c, h, h, k, r, s, p).startswith("matrix cores")
    assert not grad(8, 64, 512, 4, 1, 1, 0)     # 207, 226
    assert grad(8, 64, 112, 16, 1, 1, 0)        # 28, 22
    assert grad(64, 64, 56, 5, 3, 2, 1)         # phases together: 98, 40
