// The shift operators on the matrix cores (mfma_conv.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "conv_plan.hpp"

namespace ds {

// How a problem runs there: the packed copy of its input, its weight matrices and
// its grid. Host only; touches no device.
struct MfmaLayout {
    bool fits = false;
    bool sampled = false;        // a 1 x 1 window: the packed copy holds the sampled pixels only
    int US = 1;                  // tap columns folded into the channels of the packed copy
    int CB = 0, even = 0;        // 32-channel blocks, whether their number is even
    int nchunks = 0, tiles_p = 0, tiles_k = 0, splits = 1, cps = 0;
    int PH = 0, PW = 0, NP = 0, nblk = 0;
    size_t xp_bytes = 0, dig_bytes = 0, hm_bytes = 0, wa_bytes = 0, bd_bytes = 0;
    size_t input_bytes() const { return xp_bytes + dig_bytes + hm_bytes; }
    size_t weight_bytes() const { return wa_bytes + bd_bytes; }
};

// `shared`: the packed copy is one of all of x, usable by several problems on it;
// `tasks`: problems that share the launch (a smaller one is split less then).
MfmaLayout mfma_layout(const ConvGeom &g, bool shared = false, int tasks = 1);

// Whether the matrix cores are expected to run a problem of this many terms
// faster than the vector kernels,
bool mfma_prefer(const ConvGeom &g, int64_t terms);
// unless its reduction is so short that most of a chunk is padding. `gradient`: the
// vector kernels run it as a gradient's single phase.
bool mfma_padded(const ConvGeom &g, const MfmaLayout &l, bool gradient);

// Where a problem's weights are in the packed codes. Element (output channel k,
// reduction channel c, tap (r, s)) is the code of row k and column
// (c * R + r0 + r * dr) * S + s0 + s * ds, or with `adjoint` (input gradients)
// of row c and column (k * R + ..) * S + ...
struct MfmaWeights {
    int R = 1, S = 1, r0 = 0, dr = 1, s0 = 0, ds = 1;
    bool adjoint = false;
    int wpr = 0, bits = 5;
};
MfmaWeights mfma_forward_weights(const ConvGeom &g);
MfmaWeights mfma_phase_weights(const ConvGeom &forward, const GradPhase &phase);

// One of up to kMfmaTasks problems on one input, run in one launch.
constexpr int kMfmaTasks = 4;
struct MfmaTask {
    ConvGeom g;
    OutMap map;
    MfmaLayout l;
    MfmaWeights w;
    unsigned char *weights = nullptr;   // l.weight_bytes()
};

// First launch: packs x (act_bytes-byte integers; none when x is NULL) into
// `input` (l.input_bytes(), the layout of the first task), expands the packed
// codes wp into each task's weights (not when wp is NULL), and starts the outputs
// of split tasks at the bias. Second launch: the products, y and the epilogue.
hipError_t mfma_prepare(const MfmaTask *tasks, int ntasks, const void *x, int act_bytes, const uint32_t *wp,
                        unsigned char *input, const int32_t *bias, int32_t *y, hipStream_t st);
hipError_t mfma_multiply(const MfmaTask *tasks, int ntasks, const unsigned char *input, const int32_t *bias,
                         int32_t *y, const Epilogue &epi, hipStream_t st);


// The input gradient of forward layer g as tasks on one packed copy of dy, one per
// stride phase that a tap reaches (`zeros`: some positions of dx none reaches);
// false when a phase has no layout. `terms`: of all phases.
bool mfma_gradient_tasks(const ConvGeom &g, std::vector<MfmaTask> &tasks, bool &zeros, int64_t &terms);

// Expected duration (us) of a plan's tasks on an input of x_elems elements, the
// weights expanded when the plan is made.
double mfma_plan_us(const MfmaTask *tasks, size_t ntasks, int64_t x_elems);

}  // namespace ds
