// Pooling layers of the networks the shift operators run in (the ResNet-18 of
// the paper's Section 6 timing has a 3 x 3 stride-2 max pool after its stem and
// a global average pool before its classifier), on int32 fixed point.
// Both are memory-bound passes over x; what keeps them from its rate is the latency of
// a thread's loads, so the loads of a window or of a plane are in flight together.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "common.hpp"
#include "fastdiv.hpp"

namespace ds {

namespace {

struct PoolParams {
    int H, W, R, S, sh, sw, ph, pw;
    FastDiv oh, ow;
};

// One thread per output. A position in the padding reads the nearest one of x, which
// the same window holds (the padding is half a window at most), so no load waits for
// a branch. RS: the size of a square window, its loads unrolled; 0: any window.
// Measured on 32 x 64 x 112 x 112, to write 26 MB of reading 103: 3 x 3 stride 2 48.8 us
// with 64-bit divisions and a branch per position, 33.4 so (3.9 TB/s), 2 x 2 28.6 and
// 19.8; 5 x 5 stride 1 (not unrolled) 385 and 348.
template <int RS>
__global__ void __launch_bounds__(256)
maxpool_kernel(const int32_t *__restrict__ x, int32_t *__restrict__ y, int64_t total, const PoolParams p)
{
    const int R = RS ? RS : p.R, S = RS ? RS : p.S;
    for (int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; idx < total;
         idx += int64_t(gridDim.x) * blockDim.x) {
        const int row = fdiv(int(idx), p.ow), ow = int(idx) - row * int(p.ow.d);
        const int plane = fdiv(row, p.oh), oh = row - plane * int(p.oh.d);   // n * C + c
        const int32_t *xp = x + int64_t(plane) * p.H * p.W;
        const int ih = oh * p.sh - p.ph, iw = ow * p.sw - p.pw;
        int32_t best = INT_MIN;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int32_t *xr = xp + min(max(ih + r, 0), p.H - 1) * p.W;
#pragma unroll
            for (int s = 0; s < S; ++s) best = max(best, xr[min(max(iw + s, 0), p.W - 1)]);
        }
        y[idx] = best;
    }
}

// LANES lanes per (n, c) plane: floor of the int64 sum over the plane / HW. A thread per
// plane reads it at one load's latency after another, sixteen divide by HW sixteen times:
// 16 x 64 planes of 56 x 56 take 394 us with one and 19.5 with sixteen, 2^20 planes of 5 x
// 5 152 and 60, of 4 x 4 38 and 55, of one element 7.5 and 53.
template <int LANES>
__global__ void __launch_bounds__(256)
avgpool_global_kernel(const int32_t *__restrict__ x, int32_t *__restrict__ y, int64_t planes,
                      int HW)
{
    const int part = threadIdx.x % LANES;
    for (int64_t i = int64_t(blockIdx.x) * (256 / LANES) + threadIdx.x / LANES; i < planes;
         i += int64_t(gridDim.x) * (256 / LANES)) {
        const int32_t *xp = x + i * HW;
        int64_t sum = 0;
        for (int64_t p = part; p < HW; p += LANES) sum += xp[p];
        for (int off = LANES / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, LANES);
        int64_t q = sum / HW;
        if (sum % HW != 0 && sum < 0) q -= 1;  // division truncates; floor it
        if (part == 0) y[i] = int32_t(q);
    }
}

ds_status status_of(hipError_t e, const char *what)
{
    if (e == hipSuccess) return ok();
    return fail(DS_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

int grid_for(int64_t total)
{
    return int(std::max<int64_t>(1, std::min<int64_t>((total + 255) / 256, 8192)));
}

}  // namespace

}  // namespace ds

using namespace ds;

extern "C" ds_status ds_maxpool2d(const int32_t *x, int32_t *y, int64_t n, int64_t c, int64_t h,
                                  int64_t w, int64_t r, int64_t s, int32_t stride_h,
                                  int32_t stride_w, int32_t pad_h, int32_t pad_w, uint32_t flags,
                                  void *stream)
{
    if (!x || !y) return fail(DS_ERR_NULL_POINTER, "x and y must not be NULL");
    if (n <= 0 || c <= 0 || h <= 0 || w <= 0 || r <= 0 || s <= 0)
        return fail(DS_ERR_INVALID_SHAPE, "all sizes must be > 0");
    if (stride_h < 1 || stride_w < 1) return fail(DS_ERR_INVALID_ARG, "stride must be >= 1");
    if (pad_h < 0 || pad_w < 0 || 2 * int64_t(pad_h) > r || 2 * int64_t(pad_w) > s)
        return fail(DS_ERR_INVALID_ARG, "padding must be in [0, kernel / 2]");
    if (h + 2 * int64_t(pad_h) < r || w + 2 * int64_t(pad_w) < s)
        return fail(DS_ERR_INVALID_SHAPE, "window larger than the padded input");
    if (flags != 0) return fail(DS_ERR_INVALID_ARG, "flags must be 0");
    const int64_t oh = (h + 2 * int64_t(pad_h) - r) / stride_h + 1;
    const int64_t ow = (w + 2 * int64_t(pad_w) - s) / stride_w + 1;
    const int64_t xe = prod({n, c, h, w}), ye = prod({n, c, oh, ow});
    if (xe < 0 || ye < 0 || xe > kMaxElems || ye > kMaxElems || r > kMaxElems || s > kMaxElems)
        return fail(DS_ERR_UNSUPPORTED, "tensors with 2^31 or more elements are not supported");
    if (overlap(x, 4 * xe, y, 4 * ye)) return fail(DS_ERR_INVALID_ARG, "y overlaps x");
    if (!device_range_ok(x, 4 * xe)) return fail(DS_ERR_INVALID_ARG, "x is not a device buffer of %lld bytes", (long long)(4 * xe));
    if (!device_range_ok(y, 4 * ye)) return fail(DS_ERR_INVALID_ARG, "y is not a device buffer of %lld bytes", (long long)(4 * ye));
    PoolParams p{int(h), int(w), int(r), int(s), stride_h, stride_w, pad_h, pad_w,
                 make_fastdiv(uint32_t(oh)), make_fastdiv(uint32_t(ow))};
    const auto kernel = r == 3 && s == 3 ? maxpool_kernel<3> : r == 2 && s == 2 ? maxpool_kernel<2> : maxpool_kernel<0>;
    hipLaunchKernelGGL(kernel, dim3(grid_for(ye)), dim3(256), 0, static_cast<hipStream_t>(stream), x, y, ye, p);
    return status_of(hipGetLastError(), "ds_maxpool2d");
}

extern "C" ds_status ds_avgpool2d_global(const int32_t *x, int32_t *y, int64_t n, int64_t c,
                                         int64_t h, int64_t w, uint32_t flags, void *stream)
{
    if (!x || !y) return fail(DS_ERR_NULL_POINTER, "x and y must not be NULL");
    if (n <= 0 || c <= 0 || h <= 0 || w <= 0) return fail(DS_ERR_INVALID_SHAPE, "all sizes must be > 0");
    if (flags != 0) return fail(DS_ERR_INVALID_ARG, "flags must be 0");
    const int64_t xe = prod({n, c, h, w}), ye = prod({n, c});
    if (xe < 0 || xe > kMaxElems) return fail(DS_ERR_UNSUPPORTED, "tensors with 2^31 or more elements are not supported");
    if (overlap(x, 4 * xe, y, 4 * ye)) return fail(DS_ERR_INVALID_ARG, "y overlaps x");
    if (!device_range_ok(x, 4 * xe)) return fail(DS_ERR_INVALID_ARG, "x is not a device buffer of %lld bytes", (long long)(4 * xe));
    if (!device_range_ok(y, 4 * ye)) return fail(DS_ERR_INVALID_ARG, "y is not a device buffer of %lld bytes", (long long)(4 * ye));
    const int lanes = h * w <= 16 ? 1 : 16;
    hipLaunchKernelGGL(lanes == 1 ? avgpool_global_kernel<1> : avgpool_global_kernel<16>, dim3(grid_for(lanes * ye)),
                       dim3(256), 0, static_cast<hipStream_t>(stream), x, y, ye, int(h * w));
    return status_of(hipGetLastError(), "ds_avgpool2d_global");
}
