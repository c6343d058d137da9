// The shift operators on the matrix cores of gfx950.
//
// A right shift is not a multiplication, but it is linear in the bits of its
// operand: for x = sum_b x_b 2^b (bit 31 counting -2^31),
//     x >> s = sum_{b >= s} x_b 2^(b - s)            (floor, for every int32)
// so the shift-accumulate of a whole layer is a sum of matrix products, one per
// slice of the bits of x, whose weight matrices hold +-2^(b - s) where the
// weight's shift s lets the slice through and 0 where it does not. Slices and
// weights fit 4- and 6-bit floats exactly, products and sums are exact integers
// (bounded below 2^24 units, see `Bounds`), and the f8f6f4 matrix instructions run
// those formats at 4.4 P multiply-adds/s here (32x32x64, measured), twice their
// 8-bit rate: 20 of them make one dense shift-accumulate, 0.22 P SAC/s, against
// 17.8 T SAC/s for the two vector instructions per term of the tiled kernel.
//
// The 20 products of a 32-row by 32-pixel tile over 64 reduction elements
// (d(b) is the 2-bit digit of bits b, b+1; H = x >> 16):
//     P_b  x d(b)      b = 0, 2, 4, 6, 8: shifts 0..b; b = 10, 12, 14: shifts 6..b
//     S_b  x bit b     b = 1, 3, .. 13: shift b alone (bit b of d(b-1))
//     P_14 x H         shifts 6..14 of the high part
//     W    x d(10), d(12), d(14), H      shifts 0..5 of what lies above bit 9
// E3M2 holds the nine powers 2^-4 .. 2^4, which is why the shifts are cut at 6:
// every slot's weights span at most 2^0 .. 2^8. Weights are E3M2 (P_2 .. P_14, W)
// or E2M1 (P_0, S_b, one magnitude each); digits are E2M1, cut out of a nibble
// plane of x by one AND; H is E2M3, exact for |H| <= 16. Two float accumulators
// hold the sum: C0 in units of 1 and C1, the part of the shifts 0..5 above bit
// 11, in units of 2^7. H outside -16 .. 15 is split into four signed base-32
// digits h0 .. h3; h0 takes H's place and the three others get passes of their
// own, which a tile runs only when its images need them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>

#include "conv_plan.hpp"
#include "fastdiv.hpp"
#include "mfma_conv.hpp"

namespace ds {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;

constexpr int kBlockK = 32;          // reduction elements per lane: 32 channels of one tap
constexpr int kRows = 64;            // output channels per workgroup
constexpr int kPix = 256;            // output pixels per workgroup (64 per wave)
constexpr int kFp6 = 8, kFp4 = 8;    // weight matrices of each format
constexpr int kTileBytes = kFp6 * 1536 + kFp4 * 1024;  // one 32-row tile, 64 reduction elements
constexpr int kStageBytes = 2 * kTileBytes;            // a workgroup's 64 rows
constexpr int kXpBytes = 88;         // per pixel and 32 channels: 4 nibble planes, h0
constexpr int kDigBytes = 72;        // the same for h1, h2, h3
constexpr int kOutPitch = 65;         // LDS words per pixel of the output tile
constexpr uint32_t kOOB = 0x80000000u;
constexpr int kRsrcWord3 = 0x00020000;
constexpr int kLimit = (1 << 24) - 1;  // a float sum of integers stays exact up to 2^24

// fp6 matrices, in this order; fp4 matrices: P_0, S_1, S_3, .. S_13.
enum Fp6 { kP2, kP4, kP6, kP8, kP10, kP12, kP14, kW };

// Offset of a lane's share of matrix `i` of row tile `mt` in a stage: the first 16
// bytes (64 lanes in a row), then for fp6 8 more (lane l's at place l ^ mt: were the
// two row tiles' a fixed distance apart, one instruction would read both into
// neighbouring registers, and every one would be moved next to its first half).
__host__ __device__ constexpr int fp6_lo(int i, int mt) { return (i * 2 + mt) * 1536; }
__host__ __device__ constexpr int fp6_hi(int i, int mt) { return (i * 2 + mt) * 1536 + 1024; }
__host__ __device__ constexpr int fp4_at(int i, int mt) { return kFp6 * 2 * 1536 + (i * 2 + mt) * 1024; }

// E3M2 code of 2^(e - 4), e = 0 .. 8.
__host__ __device__ constexpr uint32_t e3m2(int e) { return e == 0 ? 1u : e == 1 ? 2u : uint32_t(e - 1) << 2; }

// Shift s's entry of fp6 matrix i, without the sign (0: the shift is not in it).
__host__ __device__ constexpr uint32_t fp6_code(int i, int s)
{
    if (s > 14) return 0u;
    if (i == kW) return s <= 5 ? e3m2(6 - s) : 0u;
    const int b = 2 * i + 2;
    return s <= b && (b <= 8 || s >= 6) ? e3m2(b - s) : 0u;
}

// Shift s's entry of fp4 matrix i: +-1.0 in P_0 (shift 0), +-0.5 in S_b (shift b).
__host__ __device__ constexpr uint32_t fp4_code(int i, int s)
{
    if (i == 0) return s == 0 ? 2u : 0u;
    return s == 2 * i - 1 ? 1u : 0u;
}

// What a chunk of 64 reduction elements can add to a row's accumulators, in their
// units, as the largest over the 32 rows of a tile (two entries per chunk): C0 by at most p0 + (hm + 1) * q0, C1 by
// r1 * (15 + 16 * hm), for |h0| <= hm. A tile converts its sums to integers before
// a bound could pass 2^24; for the weights and inputs of trained layers that is
// never before the end of up to 4608 elements, in the worst case after 960.
struct Bounds {
    int p0, q0, r1, pad;
};

struct Reduction {
    int CB;        // blocks of 32 channels
    int R, S;      // taps
    int US;        // columns of a tap row folded into the channels (1: none)
    int C;         // channels of the packed copy (US times the layer's)
    int even;      // CB even: a chunk's two blocks are two channel blocks of one tap
    int nchunks;
};

// Block (tap r, s; channel block cb) of a lane half of chunk ch.
__device__ __forceinline__ void block_at(const Reduction &d, int ch, int half, int &cb, int &r, int &s)
{
    const int taps = d.R * d.S;
    int tap;
    if (d.even) {
        cb = ch / taps;
        tap = ch - cb * taps;
        cb = 2 * cb + half;
    } else {
        const int kb = 2 * ch + half;
        cb = kb / taps;
        tap = kb - cb * taps;
    }
    r = tap / d.S;
    s = tap - r * d.S;
}

// ---------------------------------------------------------------------------
// Preparation: the weight matrices of every 64 rows and 64 reduction elements,
// one workgroup each (blocks [0, wblocks)), and the packed copy of x (the rest).

struct PackParams {
    // The packed copy's pixels (n, i, j) and where they come from: x row i * sh,
    // column j * sw - pw + the tap column folded into the channel.
    int N, C, H, W, HW;          // x
    int PH, PW, NP, PHW;         // the packed copy
    int sh, sw, pw, US;
    int CB, nblk;
    int64_t xstride_n;
    FastDiv div_phw, div_pw, div_us;
};

__device__ __forceinline__ void put6(uint32_t (&o)[6], int e, uint32_t v)
{
    const int bit = 6 * e, w = bit >> 5, sh = bit & 31;
    o[w] |= v << sh;
    if (sh > 26) o[w + 1] |= v >> (32 - sh);
}

// The weight matrices of 32 rows and 64 reduction elements (block: row block, chunk,
// row tile) and their bounds. The codes are decoded once into LDS; then each of four
// groups of 64 threads builds two fp6 and two fp4 matrices, a thread the 32 weights
// of one lane's share.
__device__ void prep_weights(const uint32_t *__restrict__ wp, int K, int R, int S, int wpr, const CodeFmt &fmt,
                             const Reduction &d, int block, unsigned char *__restrict__ wa,
                             Bounds *__restrict__ bounds)
{
    constexpr int kPitch = 80;   // bytes per row of codes: 16-byte reads, spread over the banks
    __shared__ uint32_t lut[4][32];
    __shared__ __align__(16) unsigned char codes[32][kPitch];
    const int tid = threadIdx.x, group = tid >> 6, lane = tid & 63, half = lane >> 5;
    const int unit = block >> 1, mt = block & 1;
    const int mblk = unit / d.nchunks, ch = unit - mblk * d.nchunks;
    if (tid < 128) {
        // A code's entries in a group's four matrices: 6 + 6 + 4 + 4 bits.
        const int g = tid >> 5, code = tid & 31, s = code & 15, neg = code >> 4;
        uint32_t v = 0;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t a = fp6_code(2 * g + i, s), b = fp4_code(2 * g + i, s);
            v |= (a && neg ? a | 32u : a) << (6 * i);
            v |= (b && neg ? b | 8u : b) << (12 + 4 * i);
        }
        lut[g][code] = v;
    }
    {
        // Eight codes per thread: row tid / 8, elements 8 (tid % 8) .. of one block.
        const int row = tid >> 3, seg = tid & 7, k = mblk * kRows + mt * 32 + row;
        int cb, r, s;
        block_at(d, ch, seg >> 2, cb, r, s);
        const uint32_t *wrow = wp + int64_t(min(k, K - 1)) * wpr;
        uint32_t c8[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = cb * kBlockK + (seg & 3) * 8 + e;
            int col = (c * R + r) * S + s;
            if (d.US > 1) {
                const int cl = c / d.US;
                col = (cl * R + r) * S + (c - cl * d.US);
            }
            const bool ok = k < K && cb < d.CB && c < d.C;
            const uint32_t code = fmt.at(wrow, ok ? col : 0);
            c8[e] = ok ? code : 15u;
        }
        v2i w{};
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e >> 2] |= int(c8[e] << (8 * (e & 3)));
        *reinterpret_cast<v2i *>(&codes[row][seg * 8]) = w;
    }
    __syncthreads();
    v4i cw[2];
    cw[0] = *reinterpret_cast<const v4i *>(&codes[lane & 31][half * 32]);
    cw[1] = *reinterpret_cast<const v4i *>(&codes[lane & 31][half * 32 + 16]);
    uint32_t o6[2][6] = {}, o4[2][4] = {};
    int p0 = 0, q0 = 0, r1 = 0;
#pragma unroll
    for (int e = 0; e < kBlockK; ++e) {
        const uint32_t code = (uint32_t(cw[e >> 4][(e >> 2) & 3]) >> (8 * (e & 3))) & 31u;
        const uint32_t v = lut[group][code];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            put6(o6[i], e, (v >> (6 * i)) & 63u);
            o4[i][e >> 3] |= ((v >> (12 + 4 * i)) & 15u) << (4 * (e & 7));
        }
        if (group == 0) {
            const int sft = int(code & 15u);
            p0 += sft <= 5 ? 4095 >> sft : 0;
            r1 += sft <= 5 ? 32 >> sft : 0;
            q0 += sft >= 6 && sft < 15 ? 65536 >> sft : 0;
        }
    }
    unsigned char *st = wa + int64_t(unit) * kStageBytes;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = 2 * group + i;
        *reinterpret_cast<v4i *>(st + fp6_lo(m, mt) + lane * 16) =
            v4i{int(o6[i][0]), int(o6[i][1]), int(o6[i][2]), int(o6[i][3])};
        *reinterpret_cast<v2i *>(st + fp6_hi(m, mt) + (lane ^ mt) * 8) = v2i{int(o6[i][4]), int(o6[i][5])};
        *reinterpret_cast<v4i *>(st + fp4_at(m, mt) + lane * 16) =
            v4i{int(o4[i][0]), int(o4[i][1]), int(o4[i][2]), int(o4[i][3])};
    }
    if (group == 0) {
        // A row's two halves together, then the largest over the rows.
        p0 += __shfl_xor(p0, 32);
        q0 += __shfl_xor(q0, 32);
        r1 += __shfl_xor(r1, 32);
        for (int off = 16; off > 0; off >>= 1) {
            p0 = max(p0, __shfl_xor(p0, off));
            q0 = max(q0, __shfl_xor(q0, off));
            r1 = max(r1, __shfl_xor(r1, off));
        }
        if (lane == 0) bounds[block] = Bounds{p0, q0, r1, 0};
    }
}

// E2M3 code of h / 8 for |h| <= 16.
__device__ __forceinline__ uint32_t e2m3(int h) { return h < 0 ? uint32_t(-h) | 32u : uint32_t(h); }

// The packed copy of 32 channels of 256 pixels, one pixel per lane: four planes of
// nibbles (bits 4p .. 4p+3 of the 32 channels, channel e in nibble e) and h0; h1
// .. h3 where some H of the block needs them. hmax[cb][block]: the largest |H|, or
// 255 when one lies outside -16 .. 15.
__device__ void pack_x(const int32_t *__restrict__ x, const PackParams &p, int block,
                       unsigned char *__restrict__ xp, unsigned char *__restrict__ dig,
                       unsigned char *__restrict__ hmax)
{
    __shared__ int red[4];
    const int cb = block / p.nblk, pb = block - cb * p.nblk;
    const int pix = pb * 256 + int(threadIdx.x);
    const bool in = pix < p.NP;
    const int pc = min(pix, p.NP - 1);
    const int n = fdiv(pc, p.div_phw), rem = pc - n * p.PHW;
    const int i = fdiv(rem, p.div_pw), j = rem - i * p.PW;
    const int64_t base = int64_t(n) * p.C * p.HW + int64_t(i) * p.sh * p.W + j * p.sw - p.pw;
    // Loads past the last channel (or, with folded tap columns, outside the row) are
    // redirected to a valid element and replaced by 0: no branch around any of them.
    int32_t v[kBlockK];
    const int c0 = cb * kBlockK;
    if (p.US > 1) {
#pragma unroll
        for (int e = 0; e < kBlockK; ++e) {
            const int cc = c0 + e, c = min(fdiv(cc, p.div_us), p.C - 1), s = cc - fdiv(cc, p.div_us) * p.US;
            const int col = j * p.sw - p.pw + s, cl = min(max(col, 0), p.W - 1);
            v[e] = x[base + int64_t(c) * p.HW + (cl - (j * p.sw - p.pw))];
            if (cc >= p.C * p.US || cl != col) v[e] = 0;
        }
    } else {
        if (p.HW == 1 && c0 + kBlockK <= p.C && (p.C & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0) {
            // Row-major inputs of a LinearShift: the 32 channels are consecutive.
            const v4i *src = reinterpret_cast<const v4i *>(x + base + c0);
#pragma unroll
            for (int e = 0; e < kBlockK / 4; ++e) {
                const v4i q = src[e];
#pragma unroll
                for (int t = 0; t < 4; ++t) v[4 * e + t] = q[t];
            }
        } else {
            const int32_t *src = x + base + int64_t(c0) * p.HW;
            const int last = p.C - 1 - c0;
#pragma unroll
            for (int e = 0; e < kBlockK; ++e) {
                v[e] = src[int64_t(min(e, last)) * p.HW];
            }
            if (last < kBlockK - 1) {
#pragma unroll
                for (int e = 0; e < kBlockK; ++e) v[e] = e <= last ? v[e] : 0;
            }
        }
    }
    int most = 0;
    uint32_t h6[6] = {};
#pragma unroll
    for (int e = 0; e < kBlockK; ++e) {
        const int h = v[e] >> 16;
        const int a = h < -16 || h > 15 ? 255 : h < 0 ? -h : h;
        most = max(most, a);
        put6(h6, e, e2m3(((h + 16) & 31) - 16));
    }
    const int64_t np = p.NP;
    unsigned char *o = xp + int64_t(cb) * np * kXpBytes;
    if (in) {
#pragma unroll
        for (int pl = 0; pl < 4; ++pl) {
            v4i w;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint32_t word = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    // Channels 8g + c and 8g + c + 4 in the two halves of one word.
                    const uint32_t pr = __builtin_amdgcn_perm(uint32_t(v[8 * g + c + 4]), uint32_t(v[8 * g + c]), 0x05040100u);
                    const uint32_t sft = pl >= c ? pr >> (4 * (pl - c)) : pr << (4 * (c - pl));
                    word |= sft & (0x000f000fu << (4 * c));
                }
                w[g] = int(word);
            }
            *reinterpret_cast<v4i *>(o + pl * np * 16 + int64_t(pix) * 16) = w;
        }
        v4i lo;
        v2i hi;
        for (int t = 0; t < 4; ++t) lo[t] = int(h6[t]);
        for (int t = 0; t < 2; ++t) hi[t] = int(h6[4 + t]);
        *reinterpret_cast<v4i *>(o + 64 * np + int64_t(pix) * 16) = lo;
        *reinterpret_cast<v2i *>(o + 80 * np + int64_t(pix) * 8) = hi;
    }
    for (int off = 32; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = most;
    __syncthreads();
    most = max(max(red[0], red[1]), max(red[2], red[3]));
    if (threadIdx.x == 0) hmax[block] = (unsigned char)most;
    if (most < 255 || !in) return;
#pragma unroll 1
    for (int d = 1; d < 4; ++d) {
        uint32_t q6[6] = {};
#pragma unroll
        for (int e = 0; e < kBlockK; ++e) {
            int h = v[e] >> 16, q = 0;
            for (int t = 0; t <= d; ++t) {
                q = ((h + 16) & 31) - 16;
                h = (h - q) >> 5;
            }
            put6(q6, e, e2m3(q));
        }
        unsigned char *od = dig + (int64_t(cb) * 3 + d - 1) * np * 24;
        v4i lo;
        v2i hi;
        for (int t = 0; t < 4; ++t) lo[t] = int(q6[t]);
        for (int t = 0; t < 2; ++t) hi[t] = int(q6[4 + t]);
        *reinterpret_cast<v4i *>(od + int64_t(pix) * 16) = lo;
        *reinterpret_cast<v2i *>(od + 16 * np + int64_t(pix) * 8) = hi;
    }
}

// y[n][k][oh][ow] = bias[k], where parts of the reduction are added to it.
struct FillParams {
    int32_t *y;
    const int32_t *bias;
    int K, OHOW, OW, NK, blocks;   // NK planes of OHOW elements
    int ybase, ynst, ykst, yrst, ycst;
    FastDiv div_ohow, div_ow, div_k;
};

__device__ void fill_y(const FillParams &f, int block)
{
    const int total = f.NK * f.OHOW;   // fewer than 2^31
    for (int64_t i = int64_t(block) * 256 + threadIdx.x; i < total; i += int64_t(f.blocks) * 256) {
        const int pl = fdiv(int(i), f.div_ohow), rem = int(i) - pl * f.OHOW;
        const int n = fdiv(pl, f.div_k), k = pl - n * f.K;
        const int oh = fdiv(rem, f.div_ow), ow = rem - oh * f.OW;
        f.y[int64_t(f.ybase) + int64_t(n) * f.ynst + int64_t(k) * f.ykst + int64_t(oh) * f.yrst + ow * f.ycst] =
            f.bias ? f.bias[k] : 0;
    }
}

__global__ void __launch_bounds__(256)
mfma_prep_kernel(const int32_t *__restrict__ x, const uint32_t *__restrict__ wp, int K, int R, int S,
                 int wpr, CodeFmt fmt, Reduction d, PackParams p, int wblocks,
                 unsigned char *__restrict__ wa, Bounds *__restrict__ bounds,
                 unsigned char *__restrict__ xp, unsigned char *__restrict__ dig,
                 unsigned char *__restrict__ hmax, FillParams f)
{
    const int block = int(blockIdx.x), pack = block - wblocks, fill = pack - p.CB * p.nblk;
    if (block < wblocks) prep_weights(wp, K, R, S, wpr, fmt, d, block, wa, bounds);
    else if (fill < 0) pack_x(x, p, pack, xp, dig, hmax);
    else fill_y(f, fill);
}

// ---------------------------------------------------------------------------
// The product kernel.

struct MfmaParams {
    Reduction d;
    int PH, PW, PHW, NP;            // packed copy
    int sh, sw, ph, pw;             // window placement on the packed copy
    int K, OHOW, NQ;
    int tiles_p, tiles_k, cps, nblk;
    int atomic_out, fuse_epi, rowmajor;
    int ybase, ynst, ykst, yrst, ycst;
    uint32_t xp_bytes;
    Epilogue epi;
    FastDiv div_ohow, div_ow;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, int(bytes), kRsrcWord3);
}

__device__ __forceinline__ v8i wide(v4i lo, v2i hi)
{
    return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], 0, 0};
}

__device__ __forceinline__ v8i wide(v4i lo) { return v8i{lo[0], lo[1], lo[2], lo[3], 0, 0, 0, 0}; }

// Formats of the matrix instruction. Its products take a power of two from each
// operand's block scale, 2^(v - 127): bytes of kScales, chosen by the instruction.
constexpr int kE2M3 = 2, kE3M2 = 3, kE2M1 = 4;
constexpr int kOne = 0, kM4 = 1, kP2x = 2, kP4x = 3;   // 2^0, 2^-4, 2^2, 2^4
constexpr int kScales = 127 | 123 << 8 | 129 << 16 | 131 << 24;

template <int FA, int FB>
__device__ __forceinline__ v16f mm(v8i a, v8i b, v16f c)
{
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, FA, FB, 0, 0, 0, 0);
}

template <int FA, int FB, int SA, int SB = kOne>
__device__ __forceinline__ v16f mms(v8i a, v8i b, v16f c, int scales)
{
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, FA, FB, SA, scales, SB, scales);
}

__global__ void __launch_bounds__(256, 2)
mfma_conv_kernel(const unsigned char *__restrict__ xp, const unsigned char *__restrict__ dig,
                 const unsigned char *__restrict__ hmax, const unsigned char *__restrict__ wa,
                 const Bounds *__restrict__ bounds, const int32_t *__restrict__ bias,
                 int32_t *__restrict__ y, const MfmaParams p)
{
    __shared__ __align__(16) unsigned char lds[2 * kStageBytes];
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    // Blocks are dealt to the 8 XCDs in turn: each XCD takes an eighth of the tiles, all
    // row blocks of a pixel tile one after the other, so that they read its inputs
    // through one L2.
    const int at = (int(blockIdx.x) & 7) * int(gridDim.x >> 3) + int(blockIdx.x >> 3);
    if (at >= p.tiles_p * p.tiles_k) return;
    const int tp = at / p.tiles_k, mblk = at - tp * p.tiles_k;
    const int ch0 = int(blockIdx.y) * p.cps, ch1 = min(p.d.nchunks, ch0 + p.cps);
    const int CB = p.d.CB, R = p.d.R, S = p.d.S;

    // Where the windows of this lane's two pixels start in the packed copy: the pixel
    // and its row and column (16 bits each; a row no tap can bring inside for a pixel
    // past the last).
    int pb[2], at0[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int q = tp * kPix + wave * 64 + t * 32 + (lane & 31);
        const int qc = min(q, p.NQ - 1);
        const int n = fdiv(qc, p.div_ohow), rem = qc - n * p.OHOW;
        const int oh = fdiv(rem, p.div_ow), ow = rem - oh * int(p.div_ow.d);
        const int ih = oh * p.sh - p.ph, iw = ow * p.sw - p.pw;
        pb[t] = n * p.PHW + ih * p.PW + iw;
        at0[t] = int(uint32_t(q < p.NQ ? ih : -32768) << 16) | (iw & 0xffff);
    }
    // Pixel of tap (r, s) in the packed copy, or -1 outside it.
    auto pixel = [&](int t, int r, int s) {
        const int ih = (at0[t] >> 16) + r, iw = int(int16_t(at0[t])) + s;
        return unsigned(ih) < unsigned(p.PH) && unsigned(iw) < unsigned(p.PW) ? pb[t] + r * p.PW + s : -1;
    };
    const __amdgpu_buffer_rsrc_t xr = rsrc(xp, p.xp_bytes);
    const unsigned char *wrow = wa + int64_t(mblk) * p.d.nchunks * kStageBytes;
    const __amdgpu_buffer_rsrc_t wr = rsrc(wrow, uint32_t(p.d.nchunks) * uint32_t(kStageBytes));
    const int np16 = p.NP * 16, np64 = p.NP * 64, np80 = p.NP * 80, cbs = p.NP * kXpBytes;

    // The lane half's block of the next chunk to load, advanced block by block.
    int cb, r, s;
    auto seek = [&](int ch) { block_at(p.d, ch, half, cb, r, s); };
    auto step = [&]() {
        ++s;
        if (s == S) {
            s = 0;
            ++r;
            if (r == R) {
                r = 0;
                cb += p.d.even ? 2 : 1;
            }
        }
    };
    uint32_t off[2], base;   // byte of the pixel in a plane of 16-byte entries; of the block
    auto place = [&]() {
        base = uint32_t(cb) * uint32_t(cbs);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int pix = pixel(t, r, s);
            off[t] = pix >= 0 && cb < CB ? base + uint32_t(pix) * 16u : kOOB;
        }
    };
    v4i xw[2][4], xl[2];
    v2i xh[2];
    auto load_plane = [&](int pl) {
#pragma unroll
        for (int t = 0; t < 2; ++t) xw[t][pl] = __builtin_amdgcn_raw_buffer_load_b128(xr, off[t], pl * np16, 0);
    };
    auto load_h = [&]() {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            xl[t] = __builtin_amdgcn_raw_buffer_load_b128(xr, off[t], np64, 0);
            xh[t] = __builtin_amdgcn_raw_buffer_load_b64(xr, off[t] == kOOB ? kOOB : (off[t] + base) >> 1, np80, 0);
        }
    };
    auto stage = [&](int ch, int buf) {
        const uint32_t from = uint32_t(ch) * uint32_t(kStageBytes), mine = uint32_t(wave * 1024 + lane * 16);
#pragma unroll
        for (int i = 0; i < kStageBytes / 4096; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (lds_ptr_t)(lds + buf * kStageBytes + i * 4096 + wave * 1024),
                                                     16, mine, from + uint32_t(i) * 4096u, 0, 0);
    };

    v16f c0[2][2], c1[2][2];
    auto clear = [&]() {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) c0[m][t][i] = c1[m][t][i] = 0.0f;
    };
    // The sums so far into y, `shift` bits up: stored, or added to what an earlier
    // call of the same lane stored (`more`); `last` adds the bias and the epilogue.
    // They pass through the wave's own part of the LDS, so that a store takes 64
    // consecutive pixels of one channel and the channel's parameters are scalars.
    auto flush = [&](bool more, bool last, int shift) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();   // nobody reads or fills the staged weights any more
        int32_t *out = reinterpret_cast<int32_t *>(lds) + wave * 64 * kOutPitch;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        out[(t * 32 + (lane & 31)) * kOutPitch + m * 32 + g * 8 + half * 4 + i] =
                            int(uint32_t(int(c0[m][t][g * 4 + i] * 32.0f)) +
                                (uint32_t(int(c1[m][t][g * 4 + i] * 16.0f)) << 7));
        // Written and read back by the same wave, whose LDS accesses run in order.
        __builtin_amdgcn_wave_barrier();
        // Sixteen outputs a lane at a time: the channels of one pixel (64 consecutive
        // pixels a store), or, where y holds a pixel's channels in a row (LinearShift),
        // the pixels of one channel.
        const bool byrow = p.rowmajor;
        const int q0 = tp * kPix + wave * 64, kb = mblk * kRows;
        const int q = min(q0 + (byrow ? 0 : lane), p.NQ - 1);
        const int n = fdiv(q, p.div_ohow), rem = q - n * p.OHOW;
        const int oh = fdiv(rem, p.div_ow), ow = rem - oh * int(p.div_ow.d);
        int64_t o = int64_t(p.ybase) + int64_t(n) * p.ynst + oh * p.yrst + ow * p.ycst +
                    int64_t(kb + (byrow ? lane : 0)) * p.ykst;
        const int64_t ostep = byrow ? p.ynst : p.ykst;
        const int count = byrow ? min(64, p.NQ - q0) : min(64, p.K - kb);
        const bool in = byrow ? kb + lane < p.K : q0 + lane < p.NQ;
        const int32_t *src = out + (byrow ? lane : lane * kOutPitch);
        const int sstep = byrow ? kOutPitch : 1;
        // Lane l holds the parameters of channel l of the tile.
        const bool affine = last && p.fuse_epi && p.epi.mul;
        int pbias = 0, pmul = 0, padd = 0;
        if (kb + lane < p.K) {
            if (last && bias) pbias = bias[kb + lane];
            if (affine) pmul = p.epi.mul[kb + lane];
            if (affine && p.epi.add) padd = p.epi.add[kb + lane];
        }
        const bool res = last && p.fuse_epi && p.epi.res, relu = last && p.fuse_epi && p.epi.relu;
        for (int j0 = 0; j0 < count; j0 += 16, o += 16 * ostep, src += 16 * sstep) {
            uint32_t v[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = uint32_t(src[j * sstep]) << shift;
            if (!in) continue;
            const int left = count - j0;
            if (p.atomic_out) {
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (j < left) atomicAdd(reinterpret_cast<unsigned int *>(y + o + j * ostep), v[j]);
                continue;
            }
            if (more) {
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (j < left)
                        v[j] += uint32_t(__hip_atomic_load(y + o + j * ostep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            }
            int32_t rv[16];
            if (res) {
#pragma unroll
                for (int j = 0; j < 16; ++j) rv[j] = p.epi.res[o + min(j, left - 1) * ostep];
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                v[j] += uint32_t(byrow ? pbias : __builtin_amdgcn_readlane(pbias, (j0 + j) & 63));
                if (affine) {
                    const int mul = byrow ? pmul : __builtin_amdgcn_readlane(pmul, (j0 + j) & 63);
                    const int add = byrow ? padd : __builtin_amdgcn_readlane(padd, (j0 + j) & 63);
                    v[j] = uint32_t((int64_t(int32_t(v[j])) * mul) >> p.epi.mul_shift) + uint32_t(add);
                }
                if (res) v[j] += uint32_t(rv[j]);
                if (relu && int32_t(v[j]) < 0) v[j] = 0u;
                if (j < left) y[o + j * ostep] = int32_t(v[j]);
            }
        }
    };

    const int lane8x = (lane ^ 1) * 8;
    const int sc = kScales;
    if (ch0 >= ch1) return;
    stage(ch0, 0);
    seek(ch0);
    place();
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) load_plane(pl);
    load_h();
    // Largest |H| of the images this tile reads (255: their h1 .. h3 are needed).
    int hm = 0;
    {
        const int nlo = fdiv(tp * kPix, p.div_ohow), nhi = fdiv(min(tp * kPix + kPix, p.NQ) - 1, p.div_ohow);
        const int b0 = nlo * p.PHW / 256, b1 = ((nhi + 1) * p.PHW - 1) / 256, nb = b1 - b0 + 1;
        for (int i = lane; i < nb * CB; i += 64) {
            const int cb = i / nb;
            hm = max(hm, int(hmax[cb * p.nblk + b0 + i - cb * nb]));
        }
        for (int off = 32; off > 0; off >>= 1) hm = max(hm, __shfl_xor(hm, off));
        hm = __builtin_amdgcn_readfirstlane(hm);
    }
    const bool digits = hm == 255;
    hm = min(hm, 16);

    const __amdgpu_buffer_rsrc_t dr = rsrc(dig, uint32_t(CB) * uint32_t(p.NP) * uint32_t(kDigBytes));
    const Bounds *bd = bounds + 2 * mblk * p.d.nchunks;
    // Pass 0 forms the products of the nibble planes and h0; passes 1 .. 3, for
    // inputs beyond 20 bits, those of h1, h2, h3, 5 bits further up each.
    const int passes = digits ? 4 : 1;
    int pass = 0, ch = ch0;
    bool more = false;
    for (;;) {
        clear();
        int b0 = 0, b1 = 0;
        // Chunks until the reduction ends or a sum could leave the exact range.
        const auto fits = [&](int c) {
            const Bounds u = bd[2 * c], v = bd[2 * c + 1];
            const int q0 = max(u.q0, v.q0);
            b0 += pass ? 17 * q0 : max(u.p0, v.p0) + (hm + 1) * q0;
            b1 += max(u.r1, v.r1) * (pass ? 271 : 15 + 16 * hm);
            return b0 <= kLimit && b1 <= kLimit;
        };
        if (pass == 0) {
            (void)fits(ch);
            do {
                // This wave's share of the chunk's weights has landed: only the twelve loads
                // of its inputs, issued later, may be outstanding. Behind the barrier every
                // share has, and nobody reads the other buffer any more.
                asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                stage(min(ch + 1, ch1 - 1), (ch + 1 - ch0) & 1);
                asm volatile("" ::: "memory");
                const unsigned char *buf = lds + ((ch - ch0) & 1) * kStageBytes;
                auto a6 = [&](v8i (&a)[2], int i) {
#pragma unroll
                    for (int m = 0; m < 2; ++m)
                        a[m] = wide(*reinterpret_cast<const v4i *>(buf + fp6_lo(i, m) + lane * 16),
                                    *reinterpret_cast<const v2i *>(buf + fp6_hi(i, m) + (m ? lane8x : lane * 8)));
                    __builtin_amdgcn_sched_barrier(0);
                };
                auto a4 = [&](v8i (&a)[2], int i) {
#pragma unroll
                    for (int m = 0; m < 2; ++m)
                        a[m] = wide(*reinterpret_cast<const v4i *>(buf + fp4_at(i, m) + lane * 16));
                    __builtin_amdgcn_sched_barrier(0);
                };
                // Where the next chunk's inputs are.
                if (ch + 1 < ch1) {
                    step();
                    if (!p.d.even) step();
                    place();
                } else {
                    off[0] = off[1] = kOOB;
                }
                constexpr int kDig = 0x33333333, kBit = 0x22222222;
                auto up = [&](v4i (&u)[2], int pl) {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int g = 0; g < 4; ++g) u[t][g] = int(uint32_t(xw[t][pl][g]) >> 2);
                };
                auto fp4_step = [&](const v8i (&a)[2], const v4i &d0, const v4i &d1, int mask) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        c0[m][0] = mms<kE2M1, kE2M1, kM4>(a[m], wide(d0 & mask), c0[m][0], sc);
                        c0[m][1] = mms<kE2M1, kE2M1, kM4>(a[m], wide(d1 & mask), c0[m][1], sc);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                auto fp6_step = [&](const v8i (&a)[2], const v4i &d0, const v4i &d1) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        c0[m][0] = mm<kE3M2, kE2M1>(a[m], wide(d0 & kDig), c0[m][0]);
                        c0[m][1] = mm<kE3M2, kE2M1>(a[m], wide(d1 & kDig), c0[m][1]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                // Each matrix is read one step ahead of its products; a plane's registers
                // take the next chunk's plane as soon as its last digit is cut out.
                v8i aa[2], ab[2];
                v4i u[2];
                a4(aa, 0);
                a4(ab, 1);
                fp4_step(aa, xw[0][0], xw[1][0], kDig);    // P_0
                a6(aa, kP2);
                fp4_step(ab, xw[0][0], xw[1][0], kBit);    // S_1
                a4(ab, 2);
                up(u, 0);
                load_plane(0);
                fp6_step(aa, u[0], u[1]);                  // P_2
                a6(aa, kP4);
                fp4_step(ab, u[0], u[1], kBit);            // S_3
                a4(ab, 3);
                fp6_step(aa, xw[0][1], xw[1][1]);          // P_4
                a6(aa, kP6);
                fp4_step(ab, xw[0][1], xw[1][1], kBit);    // S_5
                a4(ab, 4);
                up(u, 1);
                load_plane(1);
                fp6_step(aa, u[0], u[1]);                  // P_6
                a6(aa, kP8);
                fp4_step(ab, u[0], u[1], kBit);            // S_7
                a4(ab, 5);
                fp6_step(aa, xw[0][2], xw[1][2]);          // P_8
                a6(aa, kP10);
                fp4_step(ab, xw[0][2], xw[1][2], kBit);    // S_9
                a4(ab, 6);
                up(u, 2);
                load_plane(2);
                fp6_step(aa, u[0], u[1]);                  // P_10
                a6(aa, kW);
                fp4_step(ab, u[0], u[1], kBit);            // S_11
                a6(ab, kP12);
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        c0[m][t] = mms<kE3M2, kE2M1, kP4x>(aa[m], wide(u[t] & kDig), c0[m][t], sc);
                __builtin_amdgcn_sched_barrier(0);
                fp6_step(ab, xw[0][3], xw[1][3]);          // P_12
                a4(ab, 7);
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        c1[m][t] = mm<kE3M2, kE2M1>(aa[m], wide(xw[t][3] & kDig), c1[m][t]);
                __builtin_amdgcn_sched_barrier(0);
                fp4_step(ab, xw[0][3], xw[1][3], kBit);    // S_13
                a6(ab, kP14);
                up(u, 3);
                load_plane(3);
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        c1[m][t] = mms<kE3M2, kE2M1, kP2x>(aa[m], wide(u[t] & kDig), c1[m][t], sc);
                        c1[m][t] = mms<kE3M2, kE2M3, kP2x, kP4x>(aa[m], wide(xl[t], xh[t]), c1[m][t], sc);
                    }
                __builtin_amdgcn_sched_barrier(0);
                fp6_step(ab, u[0], u[1]);                  // P_14
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        c0[m][t] = mms<kE3M2, kE2M3, kP4x>(ab[m], wide(xl[t], xh[t]), c0[m][t], sc);
                load_h();
                __builtin_amdgcn_sched_barrier(0);
                ++ch;
            } while (ch < ch1 && fits(ch));
        } else {
            (void)fits(ch);
            do {
                v8i h[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int px = cb < CB ? pixel(t, r, s) : -1, pix = max(px, 0);
                    const bool some = px >= 0 && hmax[(px >= 0 ? cb : 0) * p.nblk + (pix >> 8)] == 255;
                    const uint32_t dbase = (uint32_t(cb) * 3u + uint32_t(pass - 1)) * uint32_t(p.NP) * 24u;
                    const v4i lo = __builtin_amdgcn_raw_buffer_load_b128(dr, some ? dbase + uint32_t(pix) * 16u : kOOB, 0, 0);
                    const v2i hi = __builtin_amdgcn_raw_buffer_load_b64(
                        dr, some ? dbase + uint32_t(np16) + uint32_t(pix) * 8u : kOOB, 0, 0);
                    h[t] = wide(lo, hi);
                }
                const unsigned char *st = wrow + int64_t(ch) * kStageBytes;
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const v8i a = wide(*reinterpret_cast<const v4i *>(st + fp6_lo(kP14, m) + lane * 16),
                                       *reinterpret_cast<const v2i *>(st + fp6_hi(kP14, m) + (lane ^ m) * 8));
                    const v8i w = wide(*reinterpret_cast<const v4i *>(st + fp6_lo(kW, m) + lane * 16),
                                       *reinterpret_cast<const v2i *>(st + fp6_hi(kW, m) + (lane ^ m) * 8));
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        c0[m][t] = mms<kE3M2, kE2M3, kP4x>(a, h[t], c0[m][t], sc);
                        c1[m][t] = mms<kE3M2, kE2M3, kP2x, kP4x>(w, h[t], c1[m][t], sc);
                    }
                }
                step();
                if (!p.d.even) step();
                ++ch;
            } while (ch < ch1 && fits(ch));
        }
        const bool end = ch == ch1;
        flush(more, end && pass + 1 == passes, 5 * pass);
        more = true;
        if (end) {
            if (++pass == passes) break;
            ch = ch0;
            seek(ch0);
        } else if (pass == 0) {
            __syncthreads();   // every wave has read its sums back
            stage(ch, (ch - ch0) & 1);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
    }
}

constexpr int64_t round256(int64_t v) { return (v + 255) & ~int64_t(255); }

}  // namespace

MfmaLayout mfma_layout(const ConvGeom &g)
{
    MfmaLayout l;
    const bool point = g.r == 1 && g.s == 1 && g.ph == 0 && g.pw == 0 &&
                       g.oh <= (g.h - 1) / g.sh + 1 && g.ow <= (g.w - 1) / g.sw + 1;
    // Few channels would leave most of a 32-channel block empty: the columns of a tap
    // row become channels instead, if that saves a third of the blocks or more.
    const int64_t plain = int64_t((g.c + kBlockK - 1) / kBlockK) * g.s;
    const int64_t folded = (int64_t(g.c) * g.s + kBlockK - 1) / kBlockK;
    l.US = !point && g.s > 1 && 3 * folded <= 2 * plain ? g.s : 1;
    l.PH = point ? g.oh : g.h;
    l.PW = point || l.US > 1 ? g.ow : g.w;
    l.CB = int((int64_t(g.c) * l.US + kBlockK - 1) / kBlockK);
    l.T = g.r * (l.US > 1 ? 1 : g.s);
    l.even = l.CB % 2 == 0;
    const int64_t np = int64_t(g.n) * l.PH * l.PW, nq = int64_t(g.n) * g.oh * g.ow;
    const int64_t nchunks = (int64_t(l.CB) * l.T + 1) / 2;
    const int64_t tiles_p = (nq + kPix - 1) / kPix, tiles_k = (g.k + kRows - 1) / kRows;
    l.xp_bytes = size_t(round256(int64_t(l.CB) * np * kXpBytes));
    l.dig_bytes = size_t(round256(int64_t(l.CB) * np * kDigBytes));
    const int64_t nblk = (np + 255) / 256;
    l.hm_bytes = size_t(round256(int64_t(l.CB) * nblk));
    l.wa_bytes = size_t(tiles_k * nchunks * kStageBytes);
    l.bd_bytes = size_t(round256(2 * tiles_k * nchunks * int64_t(sizeof(Bounds))));
    // 32-bit buffer offsets (an address past 2^31 marks a position outside x), and
    // grids of 2^31 blocks at most.
    l.fits = int64_t(l.xp_bytes) < (int64_t(1) << 31) && nchunks * kStageBytes < (int64_t(1) << 31) &&
             tiles_p * tiles_k + 8 * tiles_k < (int64_t(1) << 31) && int64_t(l.CB) * nblk + 2 * tiles_k * nchunks < (int64_t(1) << 31) &&
             int64_t(g.c) * l.US < (int64_t(1) << 30) &&
             // rows and columns in 16 bits (the extents, a window start up to a padding
             // before them, a tap up to a window after it)
             std::max(l.PH, l.PW) < 16384 && std::max(g.r, g.s) < 8192 && std::max(std::abs(g.ph), std::abs(g.pw)) < 8192;
    if (!l.fits) return l;
    l.NP = int(np);
    l.nblk = int(nblk);
    l.nchunks = int(nchunks);
    l.tiles_p = int(tiles_p);
    l.tiles_k = int(tiles_k);
    // Two workgroups fit a CU: a smaller grid splits the reduction, keeping two chunks
    // per part.
    const int64_t tiles = tiles_p * tiles_k;
    int64_t splits = 1;
    if (tiles < 384) splits = std::max<int64_t>(1, std::min<int64_t>(512 / tiles, nchunks / 2));
    l.cps = int((nchunks + splits - 1) / splits);
    l.splits = int((nchunks + l.cps - 1) / l.cps);
    return l;
}

// The vector kernels keep the smallest problems, where a call is launches and
// latency: traced on MI355X, 40 -> 65 channels 3 x 3 on 9 x 9, batch 3 (0.6 M terms)
// takes 13.0 us there and 18.6 here, 512 -> 10 on 7 x 7, batch 32 (8 M, ten of the 64
// rows of a tile in use) 15.7 and 19.7; 64 -> 64 3 x 3 on 14 x 14 (7 M) 24.1 and
// 21.4, 128 -> 128 3 x 3 on 28 x 28 (116 M) 30.6 and 22.2, and 256 -> 256 3 x 3 on
// 14 x 14 at batch 128 (14.8 G) 935 and 150. A LinearShift (256 rows or more here)
// takes five launches there: 128 -> 64 at batch 300 (2.5 M) 26.4 against 19.5.
bool mfma_prefer(const ConvGeom &g, const MfmaLayout &l)
{
    if (!l.fits) return false;
    const int64_t terms = int64_t(g.n) * g.oh * g.ow * g.k * g.crs;
    const bool linear = g.h == 1 && g.w == 1 && g.r == 1 && g.s == 1;
    return !linear && ((g.k > 16 && terms >= 4000000) || terms >= 50000000);
}

hipError_t run_mfma(const ConvGeom &g, const MfmaLayout &l, const int32_t *x, const uint32_t *wp,
                    const int32_t *bias, int32_t *y, hipStream_t st, const Epilogue &epi,
                    const OutMap &map, void *scratch)
{
    if (!l.fits) return hipErrorInvalidValue;
    unsigned char *xp = static_cast<unsigned char *>(scratch);
    unsigned char *dig = xp + l.xp_bytes;
    unsigned char *hm = dig + l.dig_bytes;
    unsigned char *wa = hm + l.hm_bytes;
    Bounds *bounds = reinterpret_cast<Bounds *>(wa + l.wa_bytes);
    const bool point = l.T == 1 && l.US == 1 && g.ph == 0 && g.pw == 0 && l.PH == g.oh && l.PW == g.ow;

    Reduction d{};
    d.CB = l.CB;
    d.R = g.r;
    d.S = l.US > 1 ? 1 : g.s;
    d.US = l.US;
    d.C = g.c * l.US;
    d.even = l.even;
    d.nchunks = l.nchunks;

    PackParams k{};
    k.N = g.n; k.C = g.c; k.H = g.h; k.W = g.w; k.HW = g.h * g.w;
    k.PH = l.PH; k.PW = l.PW; k.NP = l.NP; k.PHW = l.PH * l.PW;
    k.sh = point ? g.sh : 1;
    k.sw = point || l.US > 1 ? g.sw : 1;
    k.pw = l.US > 1 ? g.pw : 0;
    k.US = l.US;
    k.CB = l.CB;
    k.nblk = l.nblk;
    k.div_phw = make_fastdiv(uint32_t(k.PHW));
    k.div_pw = make_fastdiv(uint32_t(k.PW));
    k.div_us = make_fastdiv(uint32_t(l.US));

    const bool split = l.splits > 1;
    const OutMap m = map.dense() ? OutMap{0, g.k * g.oh * g.ow, g.oh * g.ow, g.ow, 1} : map;
    FillParams f{};
    f.y = y;
    f.bias = bias;
    f.K = g.k; f.OHOW = g.oh * g.ow; f.OW = g.ow; f.NK = g.n * g.k;
    f.ybase = int(m.base); f.ynst = m.nstride; f.ykst = m.kstride; f.yrst = m.rstride; f.ycst = m.cstride;
    f.div_ohow = make_fastdiv(uint32_t(f.OHOW));
    f.div_ow = make_fastdiv(uint32_t(f.OW));
    f.div_k = make_fastdiv(uint32_t(f.K));
    f.blocks = split ? int(std::min<int64_t>((int64_t(f.NK) * f.OHOW + 1023) / 1024, 2048)) : 0;

    const int wblocks = 2 * l.tiles_k * l.nchunks;
    hipLaunchKernelGGL(mfma_prep_kernel, dim3(unsigned(wblocks) + unsigned(l.CB) * unsigned(l.nblk) + unsigned(f.blocks)),
                       dim3(256), 0, st, x, wp, g.k, g.r, g.s, int(row_words_bits(g.crs, g.bits)), code_fmt(g.bits), d,
                       k, wblocks, wa, bounds, xp, dig, hm, f);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    MfmaParams p{};
    p.d = d;
    p.PH = l.PH; p.PW = l.PW; p.PHW = k.PHW; p.NP = l.NP;
    p.sh = point ? 1 : g.sh;
    p.sw = point || l.US > 1 ? 1 : g.sw;
    p.ph = g.ph;
    p.pw = l.US > 1 ? 0 : g.pw;
    p.K = g.k; p.OHOW = g.oh * g.ow; p.NQ = int(int64_t(g.n) * p.OHOW);
    p.tiles_p = l.tiles_p; p.tiles_k = l.tiles_k; p.cps = l.cps; p.nblk = l.nblk;
    p.atomic_out = split;
    p.fuse_epi = epi.any() && !split;
    p.ybase = int(m.base); p.ynst = m.nstride; p.ykst = m.kstride; p.yrst = m.rstride; p.ycst = m.cstride;
    p.rowmajor = m.kstride == 1 && p.OHOW == 1;
    p.xp_bytes = uint32_t(l.xp_bytes);
    p.epi = epi;
    p.div_ohow = make_fastdiv(uint32_t(p.OHOW));
    p.div_ow = make_fastdiv(uint32_t(g.ow));
    const unsigned grid = unsigned(int64_t(l.tiles_p) * l.tiles_k + 7) / 8u * 8u;
    hipLaunchKernelGGL(mfma_conv_kernel, dim3(grid, unsigned(l.splits)), dim3(256), 0, st, xp, dig, hm, wa, bounds,
                       split ? nullptr : bias, y, p);
    e = hipGetLastError();
    if (e == hipSuccess && split && epi.any()) e = run_epilogue(g, y, epi, st);
    return e;
}

}  // namespace ds
