// The shift operators on the matrix cores (mfma_conv.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "conv_plan.hpp"

namespace ds {

// How a problem runs there: the packed copy of its input, its weight matrices and
// its grid. Host only; touches no device.
struct MfmaLayout {
    bool fits = false;
    int US = 1;                  // tap columns folded into the channels of the packed copy
    int CB = 0, T = 0, even = 0; // 32-channel blocks, taps, whether CB is even
    int nchunks = 0, tiles_p = 0, tiles_k = 0, splits = 1, cps = 0;
    int PH = 0, PW = 0, NP = 0, nblk = 0;
    size_t xp_bytes = 0, dig_bytes = 0, hm_bytes = 0, wa_bytes = 0, bd_bytes = 0;
    size_t bytes() const { return xp_bytes + dig_bytes + hm_bytes + wa_bytes + bd_bytes; }
};

MfmaLayout mfma_layout(const ConvGeom &g);

// Whether the matrix cores are expected to run g (laid out as `l`) faster than
// the vector kernels.
bool mfma_prefer(const ConvGeom &g, const MfmaLayout &l);

// Enqueues y = the shift convolution of x, as run_conv does, with `scratch` of at
// least l.bytes() bytes, 256-byte aligned.
hipError_t run_mfma(const ConvGeom &g, const MfmaLayout &l, const int32_t *x, const uint32_t *wp,
                    const int32_t *bias, int32_t *y, hipStream_t st, const Epilogue &epi,
                    const OutMap &map, void *scratch);

}  // namespace ds
