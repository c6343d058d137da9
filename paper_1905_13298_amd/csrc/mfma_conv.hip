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
// own, which a tile runs only as far as the inputs that it reads need them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "common.hpp"
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
constexpr int kOutPitch = 68;         // LDS words per pixel of the output tile: 16-byte rows, no bank conflicts
constexpr int kParked = 4 * 64 * kOutPitch * 4;   // bytes of the output tile
constexpr int kDigitStage = 4 * 1536;  // P_14 and W of 64 rows, one after the other in a stage
static_assert(kParked + 2 * kDigitStage <= 2 * kStageBytes, "the parked sums and two chunks of the digit passes");
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
    int C, W, HW;                // x
    int NP, PHW;                 // the packed copy
    int sh, sw, pw, US, nblk;
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
struct WeightTask {
    Reduction d;
    MfmaWeights w;
    CodeFmt fmt;
    int K, blocks;
    unsigned char *wa;
    Bounds *bounds;
};

__device__ void prep_weights(const uint32_t *__restrict__ wp, const WeightTask &t, int block)
{
    const Reduction &d = t.d;
    constexpr int kPitch = 80;   // bytes per row of codes: 16-byte reads, spread over the banks
    __shared__ uint2 lut[4][32], sizes[32];
    __shared__ __align__(16) unsigned char codes[32][kPitch];
    const int tid = threadIdx.x, group = tid >> 6, lane = tid & 63, half = lane >> 5;
    const int unit = block >> 1, mt = block & 1;
    const int mblk = unit / d.nchunks, ch = unit - mblk * d.nchunks;
    if (tid < 128) {
        // A code's entries in a group's four matrices: two of 6 bits in the halves of x,
        // two of 4 in those of y, so that neighbours are joined for both at once. (About twelve
        // instructions a code with all four in one word, five so; the expansion of 4096 x
        // 4096 codes, 168 MB, 58.6 us then and 45.7 now.)
        const int g = tid >> 5, code = tid & 31, s = code & 15, neg = code >> 4;
        uint2 v{};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t a = fp6_code(2 * g + i, s), b = fp4_code(2 * g + i, s);
            v.x |= (a && neg ? a | 32u : a) << (16 * i);
            v.y |= (b && neg ? b | 8u : b) << (16 * i);
        }
        lut[g][code] = v;
        // Its shares of the bounds: x = p0 | r1 << 20 (32 codes stay below 2^20, 2^11).
        if (g == 0)
            sizes[code] = uint2{uint32_t(s <= 5 ? 4095 >> s | 32 >> s << 20 : 0), uint32_t(s >= 6 && s < 15 ? 65536 >> s : 0)};
    }
    {
        // Eight codes per thread: row tid / 8, elements 8 (tid % 8) .. of one block.
        const int row = tid >> 3, seg = tid & 7, k = mblk * kRows + mt * 32 + row;
        int cb, r, s;
        block_at(d, ch, seg >> 2, cb, r, s);
        const int kc = min(k, t.K - 1), tap = t.w.r0 + r * t.w.dr;
        uint32_t c8[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = cb * kBlockK + (seg & 3) * 8 + e;
            const bool ok = k < t.K && cb < d.CB && c < d.C;
            int cl = ok ? c : 0, sx = s;
            if (d.US > 1) {
                const int q = cl / d.US;
                sx = cl - q * d.US;
                cl = q;
            }
            const int prow = t.w.adjoint ? cl : kc, pch = t.w.adjoint ? kc : cl;
            const int col = ok ? (pch * t.w.R + tap) * t.w.S + t.w.s0 + sx * t.w.ds : 0;
            const uint32_t code = t.fmt.at(wp + int64_t(prow) * t.w.wpr, col);
            c8[e] = ok ? code : 15u;
        }
        v2i w{};
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e >> 2] |= int(c8[e] << (8 * (e & 3) + 3));   // times an entry's bytes
        *reinterpret_cast<v2i *>(&codes[row][seg * 8]) = w;
    }
    __syncthreads();
    v4i cw[2];
    cw[0] = *reinterpret_cast<const v4i *>(&codes[lane & 31][half * 32]);
    cw[1] = *reinterpret_cast<const v4i *>(&codes[lane & 31][half * 32 + 16]);
    uint32_t o6[2][6] = {}, o4[2][4] = {};
    auto entry = [&](const uint2 *table, int e) {
        const uint32_t byte = (uint32_t(cw[e >> 4][(e >> 2) & 3]) >> (8 * (e & 3))) & 255u;
        return *reinterpret_cast<const uint2 *>(reinterpret_cast<const unsigned char *>(table) + byte);
    };
    auto put12 = [](uint32_t (&o)[6], int pair, uint32_t v) {
        const int at = 12 * pair, sh = at & 31;
        o[at >> 5] |= v << sh;
        if (sh + 12 > 32) o[(at >> 5) + 1] |= v >> (32 - sh);
    };
#pragma unroll
    for (int e = 0; e < kBlockK; e += 8) {
        uint32_t four[2] = {};
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
            const uint2 u = entry(lut[group], e + j), v = entry(lut[group], e + j + 1);
            const uint32_t six = u.x | v.x << 6;
            put12(o6[0], (e + j) / 2, six & 0xffffu);
            put12(o6[1], (e + j) / 2, six >> 16);
            four[j >> 2] |= (u.y | v.y << 4) << (4 * (j & 2));
        }
        o4[0][e >> 3] = (four[0] & 0xffffu) | four[1] << 16;
        o4[1][e >> 3] = four[0] >> 16 | (four[1] & 0xffff0000u);
    }
    unsigned char *st = t.wa + int64_t(unit) * kStageBytes;
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
        uint32_t pr = 0;
        int q0 = 0;
#pragma unroll
        for (int e = 0; e < kBlockK; ++e) {
            const uint2 v = entry(sizes, e);
            pr += v.x;
            q0 += int(v.y);
        }
        int p0 = int(pr & 0xfffffu), r1 = int(pr >> 20);
        // A row's two halves together, then the largest over the rows.
        p0 += __shfl_xor(p0, 32);
        q0 += __shfl_xor(q0, 32);
        r1 += __shfl_xor(r1, 32);
        for (int off = 16; off > 0; off >>= 1) {
            p0 = max(p0, __shfl_xor(p0, off));
            q0 = max(q0, __shfl_xor(q0, off));
            r1 = max(r1, __shfl_xor(r1, off));
        }
        if (lane == 0) t.bounds[block] = Bounds{p0, q0, r1, 0};
    }
}

// E2M3 code of h / 8 for |h| <= 16.
__device__ __forceinline__ uint32_t e2m3(int h) { return h < 0 ? uint32_t(-h) | 32u : uint32_t(h); }

// The packed copy of 32 channels of 256 pixels, one pixel per lane: four planes of
// nibbles (bits 4p .. 4p+3 of the 32 channels, channel e in nibble e) and h0; h1
// .. h3 as far as some H of the block needs them. hmax[cb][block]: the largest |H|, or
// 252 and the last digit that an H outside -16 .. 15 needs.
template <typename T>
__device__ void pack_x(const T *__restrict__ x, const PackParams &p, int block, unsigned char *__restrict__ xp,
                       unsigned char *__restrict__ dig, unsigned char *__restrict__ hmax)
{
    __shared__ int red[4];
    const int cb = block / p.nblk, pb = block - cb * p.nblk;
    const int pix = pb * 256 + int(threadIdx.x);
    const bool in = pix < p.NP;
    const int pc = min(pix, p.NP - 1);
    const int n = fdiv(pc, p.div_phw), rem = pc - n * p.PHW;
    const int i = fdiv(rem, p.div_pw), j = rem - i * int(p.div_pw.d);
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
        if (sizeof(T) == 4 && p.HW == 1 && c0 + kBlockK <= p.C && (p.C & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0) {
            // Row-major inputs of a LinearShift: the 32 channels are consecutive.
            const v4i *src = reinterpret_cast<const v4i *>(x + base + c0);
#pragma unroll
            for (int e = 0; e < kBlockK / 4; ++e) {
                const v4i q = src[e];
#pragma unroll
                for (int t = 0; t < 4; ++t) v[4 * e + t] = q[t];
            }
        } else {
            const T *src = x + base + int64_t(c0) * p.HW;
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
    int32_t low = 0, high = 0;
    uint32_t h6[6] = {};
#pragma unroll
    for (int e = 0; e < kBlockK; ++e) {
        const int h = v[e] >> 16;
        low = min(low, v[e]);
        high = max(high, v[e]);
        put6(h6, e, e2m3(((h + 16) & 31) - 16));
    }
    low >>= 16;
    high >>= 16;
    // (two digits hold -528 .. 495, three -16912 .. 15855)
    int most = low >= -16 && high <= 15 ? max(-low, high) : low >= -528 && high <= 495 ? 253 : low >= -16912 && high <= 15855 ? 254 : 255;
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
    if (most < 253 || !in) return;
#pragma unroll 1
    for (int d = 1; d <= most - 252; ++d) {
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

struct PrepArgs {
    const void *x;
    const uint32_t *wp;
    unsigned char *xp, *dig, *hmax;
    PackParams p;
    int wblocks, pblocks;            // of all tasks together; blocks past both fill
    WeightTask w[kMfmaTasks];
    FillParams f[kMfmaTasks];
};

template <typename T>
__global__ void __launch_bounds__(256) mfma_prep_kernel(const PrepArgs a)
{
    int block = int(blockIdx.x);
    if (block < a.wblocks) {
        int i = 0;
        while (block >= a.w[i].blocks) block -= a.w[i++].blocks;
        prep_weights(a.wp, a.w[i], block);
        return;
    }
    block -= a.wblocks;
    if (block < a.pblocks) {
        pack_x(static_cast<const T *>(a.x), a.p, block, a.xp, a.dig, a.hmax);
        return;
    }
    block -= a.pblocks;
    int i = 0;
    while (block >= a.f[i].blocks) block -= a.f[i++].blocks;
    fill_y(a.f[i], block);
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
    FastDiv div_ohow, div_ow;
    const unsigned char *wa;
    const Bounds *bounds;
};

struct ProductArgs {
    const unsigned char *xp, *dig, *hmax;
    const int32_t *bias;             // of the tasks that are not split
    int32_t *y;
    Epilogue epi;
    MfmaParams p[kMfmaTasks];
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
mfma_conv_kernel(const ProductArgs a)
{
    const MfmaParams &p = a.p[blockIdx.z];
    const Epilogue &epi = a.epi;
    int32_t *const y = a.y;
    const int32_t *const bias = p.atomic_out ? nullptr : a.bias;
    const unsigned char *const hmax = a.hmax;
    __shared__ __align__(16) unsigned char lds[2 * kStageBytes];
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    // Blocks are dealt to the 8 XCDs in turn: each XCD takes an eighth of the tiles, all
    // row blocks of a pixel tile one after the other, so that they read its inputs
    // through one L2.
    const int tiles = p.tiles_p * p.tiles_k, share = (tiles + 7) >> 3, place = int(blockIdx.x >> 3);
    const int at = (int(blockIdx.x) & 7) * share + place;
    if (place >= share || at >= tiles) return;
    const int tp = at / p.tiles_k, mblk = at - tp * p.tiles_k;
    const int ch0 = int(blockIdx.y) * p.cps, ch1 = min(p.d.nchunks, ch0 + p.cps);
    const int CB = p.d.CB, R = p.d.R, S = p.d.S, PH = p.PH, PW = p.PW;

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
        return (unsigned(ih) < unsigned(PH)) & (unsigned(iw) < unsigned(PW)) ? pb[t] + r * PW + s : -1;
    };
    const __amdgpu_buffer_rsrc_t xr = rsrc(a.xp, p.xp_bytes);
    const unsigned char *wrow = p.wa + int64_t(mblk) * p.d.nchunks * kStageBytes;
    const __amdgpu_buffer_rsrc_t wr = rsrc(wrow, uint32_t(p.d.nchunks) * uint32_t(kStageBytes));
    const int np16 = p.NP * 16, np64 = p.NP * 64, np80 = p.NP * 80, cbs = p.NP * kXpBytes;

    // The lane half's block of the next chunk to load, advanced block by block.
    int cb, r, s;
    auto seek = [&](int ch) { block_at(p.d, ch, half, cb, r, s); };
    const int stride = p.d.even ? 2 : 1;
    auto step = [&]() {
        const bool row = s + 1 == S, block = row & (r + 1 == R);
        s = row ? 0 : s + 1;
        r = block ? 0 : row ? r + 1 : r;
        cb += block ? stride : 0;
    };
    uint32_t off[2], base;   // byte of the pixel in a plane of 16-byte entries; of the block
    auto locate = [&]() {
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
    // (past the last chunk: zeros from outside the buffer, so that a chunk always has
    // the same number of loads in flight)
    auto stage = [&](int ch, int buf) {
        const uint32_t from = uint32_t(ch) * uint32_t(kStageBytes), mine = uint32_t(wave * 1024 + lane * 16);
#pragma unroll
        for (int i = 0; i < kStageBytes / 4096; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (lds_ptr_t)(lds + buf * kStageBytes + i * 4096 + wave * 1024),
                                                     16, ch < ch1 ? mine : kOOB, from + uint32_t(i) * 4096u, 0, 0);
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
    // The sums so far as integers in the wave's own part of the LDS, `shift` bits up:
    // written, or added to what is there (`add`). The products of the digits h1 .. h3
    // meet those of the rest here: y, read and written again by each pass, took as long
    // as the products (64 -> 64 channels 3 x 3 on 56 x 56 at batch 128, four passes: 514 us
    // so, 309 us here, with nothing else changed; one pass takes 156).
    int32_t *const out = reinterpret_cast<int32_t *>(lds) + wave * 64 * kOutPitch;
    auto park = [&](bool add, int shift) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    v4i *const at = reinterpret_cast<v4i *>(out + (t * 32 + (lane & 31)) * kOutPitch + m * 32 + g * 8 + half * 4);
                    v4i v;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        v[i] = int((uint32_t(int(c0[m][t][g * 4 + i] * 32.0f)) +
                                    (uint32_t(int(c1[m][t][g * 4 + i] * 16.0f)) << 7)) << shift);
                    if (add) {
                        const v4i o = *at;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = int(uint32_t(v[i]) + uint32_t(o[i]));
                    }
                    *at = v;
                }
        // Written and read back by the same wave, whose LDS accesses run in order.
        __builtin_amdgcn_wave_barrier();
    };
    // They go to y: stored, or added to what an earlier call of the same lane stored
    // (`more`); `last` adds the bias and the epilogue. Through the LDS a store takes 64
    // consecutive pixels of one channel and the channel's parameters are scalars.
    auto emit = [&](bool more, bool last) {
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
        const bool affine = last && p.fuse_epi && epi.mul;
        int pbias = 0, pmul = 0, padd = 0;
        if (kb + lane < p.K) {
            if (last && bias) pbias = bias[kb + lane];
            if (affine) pmul = epi.mul[kb + lane];
            if (affine && epi.add) padd = epi.add[kb + lane];
        }
        const bool res = last && p.fuse_epi && epi.res, relu = last && p.fuse_epi && epi.relu;
        // (Conditions stand outside the loops over the sixteen: a branch per output took
        // 7 us of a tile that the stores take 2 us of.)
        for (int j0 = 0; j0 < count; j0 += 16, o += 16 * ostep, src += 16 * sstep) {
            uint32_t v[16];
            if (byrow) {
#pragma unroll
                for (int j = 0; j < 16; ++j) v[j] = uint32_t(src[j * kOutPitch]);
            } else {
#pragma unroll
                for (int j = 0; j < 16; j += 4) {
                    const v4i q = *reinterpret_cast<const v4i *>(src + j);
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[j + i] = uint32_t(q[i]);
                }
            }
            const int left = count - j0;
            int32_t *yp = y + o;
            if (p.atomic_out) {
                if (in) {
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        if (j < left) atomicAdd(reinterpret_cast<unsigned int *>(yp + j * ostep), v[j]);
                }
                continue;
            }
            // The parameters are read while every lane is there: a lane past the last
            // pixel holds a channel's too.
            int bj[16], mj[16], aj[16];
            if (bias) {
#pragma unroll
                for (int j = 0; j < 16; ++j) bj[j] = byrow ? pbias : __builtin_amdgcn_readlane(pbias, (j0 + j) & 63);
            }
            if (affine) {
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    mj[j] = byrow ? pmul : __builtin_amdgcn_readlane(pmul, (j0 + j) & 63);
                    aj[j] = byrow ? padd : __builtin_amdgcn_readlane(padd, (j0 + j) & 63);
                }
            }
            if (!in) continue;
            if (more) {
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    v[j] += uint32_t(__hip_atomic_load(yp + min(j, left - 1) * ostep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            }
            if (bias) {
#pragma unroll
                for (int j = 0; j < 16; ++j) v[j] += uint32_t(bj[j]);
            }
            if (affine) {
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    v[j] = uint32_t((int64_t(int32_t(v[j])) * mj[j]) >> epi.mul_shift) + uint32_t(aj[j]);
            }
            if (res) {
                const int32_t *rp = epi.res + o;
                int32_t rv[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) rv[j] = rp[min(j, left - 1) * ostep];
#pragma unroll
                for (int j = 0; j < 16; ++j) v[j] += uint32_t(rv[j]);
            }
            if (relu) {
#pragma unroll
                for (int j = 0; j < 16; ++j) v[j] = uint32_t(max(int32_t(v[j]), 0));
            }
            if (left >= 16) {
#pragma unroll
                for (int j = 0; j < 16; ++j, yp += ostep) *yp = int32_t(v[j]);
            } else {
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (j < left) yp[j * ostep] = int32_t(v[j]);
            }
        }
    };

    const int lane8x = (lane ^ 1) * 8;
    const int sc = kScales;
    if (ch0 >= ch1) return;   // a task with fewer parts than the launch
    // Largest |H| of the blocks of packed rows this tile reads (253 .. 255: their digits up
    // to h1 .. h3 are needed), from its first output's first row to its last one's last. The first
    // entries are fetched before everything else, so that their maximum is formed
    // while the first chunk is on its way. (Over whole images the entries grow with the
    // image: 64 -> 64 channels 3 x 3 on one of 1024 x 1024 took 620 us so, 401 here; 3 -> 16
    // on 2048 x 2048 2015 and 481.)
    const int qf = tp * kPix, nf = fdiv(qf, p.div_ohow), rf = fdiv(qf - nf * p.OHOW, p.div_ow) * p.sh - p.ph;
    const int ql = min(qf + kPix, p.NQ) - 1, nl = fdiv(ql, p.div_ohow);
    const int rl = fdiv(ql - nl * p.OHOW, p.div_ow) * p.sh - p.ph + R - 1;
    const int hb0 = (nf * p.PHW + min(max(rf, 0), p.PH - 1) * p.PW) / 256;
    const int hnb = (nl * p.PHW + min(max(rl, 0), p.PH - 1) * p.PW + p.PW - 1) / 256 - hb0 + 1;
    auto hload = [&](int i) {
        const int b = i / hnb;
        return i < hnb * CB ? int(hmax[b * p.nblk + hb0 + i - b * hnb]) : 0;
    };
    int hm = hload(lane);
    stage(ch0, 0);
    // The chunk loop waits for the staged weights by count: the twelve loads of the
    // inputs have to come after them.
    asm volatile("" ::: "memory");
    seek(ch0);
    locate();
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) load_plane(pl);
    load_h();
    const __amdgpu_buffer_rsrc_t dr = rsrc(a.dig, uint32_t(CB) * uint32_t(p.NP) * uint32_t(kDigBytes));
    const Bounds *bd = p.bounds + 2 * mblk * p.d.nchunks;
    // Pass 0 forms the products of the nibble planes and h0; passes 1 .. 3, for
    // inputs beyond 20, 25 and 30 bits, those of h1, h2, h3, 5 bits further up each.
    for (int i = lane + 64; i - lane < hnb * CB; i += 64) hm = max(hm, hload(i));
    for (int off = 32; off > 0; off >>= 1) hm = max(hm, __shfl_xor(hm, off));
    hm = __builtin_amdgcn_readfirstlane(hm);
    const int passes = hm < 253 ? 1 : hm - 251;
    hm = min(hm, 16);
    int hleast = 255;   // the least of them, where it matters
    if (passes > 1) {
        for (int i = lane; i < hnb * CB; i += 64) hleast = min(hleast, hload(i));
        for (int off = 32; off > 0; off >>= 1) hleast = min(hleast, __shfl_xor(hleast, off));
        hleast = __builtin_amdgcn_readfirstlane(hleast);
    }
    int ch = ch0, b0 = 0, b1 = 0;
    bool more = false;
    // Whether chunk c can be added before a sum could leave the exact range.
    const auto fits = [&](int c) {
        const Bounds u = bd[2 * c], v = bd[2 * c + 1];
        b0 += max(u.p0, v.p0) + (hm + 1) * max(u.q0, v.q0);
        b1 += max(u.r1, v.r1) * (15 + 16 * hm);
        return b0 <= kLimit && b1 <= kLimit;
    };
    for (;;) {
        clear();
        b0 = b1 = 0;
        (void)fits(ch);
        do {
            // This wave's share of the chunk's weights has landed: only the twelve loads
            // of its inputs, issued later, may be outstanding. Behind the barrier every
            // share has, and nobody reads the other buffer any more.
            asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            stage(ch + 1, (ch + 1 - ch0) & 1);
            asm volatile("" ::: "memory");
            const unsigned char *buf = lds + ((ch - ch0) & 1) * kStageBytes;
            auto a6 = [&](v8i (&a)[2], int i) {
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    a[m] = wide(*reinterpret_cast<const v4i *>(buf + fp6_lo(i, m) + lane * 16),
                                *reinterpret_cast<const v2i *>(buf + fp6_hi(i, m) + (m ? lane8x : lane * 8)));
            };
            auto a4 = [&](v8i (&a)[2], int i) {
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    a[m] = wide(*reinterpret_cast<const v4i *>(buf + fp4_at(i, m) + lane * 16));
            };
            // Where the next chunk's inputs are.
            if (ch + 1 < ch1) {
                step();
                if (!p.d.even) step();
                locate();
            } else {
                off[0] = off[1] = kOOB;
            }
            constexpr int kDig = 0x33333333, kBit = 0x22222222;
            // A step: the products of one matrix, the reads of the next one's share, and
            // the next digits, cut out while the products run. `region` ends it (the
            // scheduler keeps a step's instructions together: four products, with
            // vector instructions between them).
            v8i aa[2], ab[2];
            v4i d0[2], d1[2], u[2];
            auto cut = [&](v4i (&d)[2], const v4i &x0, const v4i &x1, int mask) {
                d[0] = x0 & mask;
                d[1] = x1 & mask;
            };
            auto up = [&](int pl) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int g = 0; g < 4; ++g) u[t][g] = int(uint32_t(xw[t][pl][g]) >> 2);
            };
            auto region = [&](auto products) {
                // (a count of the products the step holds, in twos of two and three
                // vector instructions)
                constexpr int n = decltype(products)::value;
                __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
                for (int i = 0; i < n; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            using Four = std::integral_constant<int, 4>;
            using Eight = std::integral_constant<int, 8>;
            auto bits = [&](const v8i (&a)[2], const v4i (&d)[2]) {     // S_b, P_0
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int t = 0; t < 2; ++t) c0[m][t] = mms<kE2M1, kE2M1, kM4>(a[m], wide(d[t]), c0[m][t], sc);
            };
            auto powers = [&](const v8i (&a)[2], const v4i (&d)[2]) {   // P_2 ..
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int t = 0; t < 2; ++t) c0[m][t] = mm<kE3M2, kE2M1>(a[m], wide(d[t]), c0[m][t]);
            };
            a4(aa, 0);
            cut(d0, xw[0][0], xw[1][0], kDig);
            __builtin_amdgcn_sched_barrier(0);
            // A plane's registers take the next chunk's plane as soon as its last digit is
            // cut out.
            auto plane = [&](auto pl_, auto first, auto last) {
                constexpr int pl = decltype(pl_)::value;
                a4(ab, 2 * pl + 1);
                if constexpr (pl == 0) bits(aa, d0);
                else powers(aa, d0);                               // P of the low digit
                cut(d1, xw[0][pl], xw[1][pl], kBit);
                region(Four());
                a6(aa, 2 * pl);
                bits(ab, d1);                                      // S of its upper bit
                up(pl);
                cut(d0, u[0], u[1], kDig);
                region(Four());
                load_plane(pl);
                first();
                powers(aa, d0);                                    // P of the high digit
                cut(d1, u[0], u[1], kBit);
                region(Four());
                last();
            };
            plane(std::integral_constant<int, 0>(), [&] { a4(ab, 2); }, [&] {
                a6(aa, kP4);
                bits(ab, d1);                                      // S_3
                cut(d0, xw[0][1], xw[1][1], kDig);
                region(Four());
            });
            plane(std::integral_constant<int, 1>(), [&] { a4(ab, 4); }, [&] {
                a6(aa, kP8);
                bits(ab, d1);                                      // S_7
                cut(d0, xw[0][2], xw[1][2], kDig);
                region(Four());
            });
            a4(ab, 5);
            powers(aa, d0);                                        // P_8
            cut(d1, xw[0][2], xw[1][2], kBit);
            region(Four());
            a6(aa, kP10);
            bits(ab, d1);                                          // S_9
            up(2);
            cut(d0, u[0], u[1], kDig);
            region(Four());
            load_plane(2);
            a4(ab, 6);
            powers(aa, d0);                                        // P_10
            cut(d1, u[0], u[1], kBit);
            region(Four());
            a6(aa, kW);
            bits(ab, d1);                                          // S_11
            cut(d1, xw[0][3], xw[1][3], kDig);
            region(Four());
            a6(ab, kP12);
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int t = 0; t < 2; ++t) {                      // W x d(10), d(12)
                    c0[m][t] = mms<kE3M2, kE2M1, kP4x>(aa[m], wide(d0[t]), c0[m][t], sc);
                    c1[m][t] = mm<kE3M2, kE2M1>(aa[m], wide(d1[t]), c1[m][t]);
                }
            region(Eight());
            cut(d0, xw[0][3], xw[1][3], kBit);
            powers(ab, d1);                                        // P_12
            up(3);
            region(Four());
            load_plane(3);
            a4(ab, 7);
            cut(d1, u[0], u[1], kDig);
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int t = 0; t < 2; ++t)                        // W x H
                    c1[m][t] = mms<kE3M2, kE2M3, kP2x, kP4x>(aa[m], wide(xl[t], xh[t]), c1[m][t], sc);
            region(Four());
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int t = 0; t < 2; ++t)                        // W x d(14)
                    c1[m][t] = mms<kE3M2, kE2M1, kP2x>(aa[m], wide(d1[t]), c1[m][t], sc);
            __builtin_amdgcn_sched_barrier(0);
            a6(aa, kP14);
            bits(ab, d0);                                          // S_13
            region(Four());
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int t = 0; t < 2; ++t)                        // P_14 x H
                    c0[m][t] = mms<kE3M2, kE2M3, kP4x>(aa[m], wide(xl[t], xh[t]), c0[m][t], sc);
            load_h();
            __builtin_amdgcn_sched_barrier(0);
            powers(aa, d1);                                        // P_14
            __builtin_amdgcn_sched_barrier(0);
            ++ch;
        } while (ch < ch1 && fits(ch));
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();   // nobody reads or fills the staged weights any more
        park(false, 0);
        if (ch == ch1) break;
        // A sum would leave the exact range: y takes what there is, the staging goes on.
        emit(more, false);
        more = true;
        __syncthreads();   // every wave has read its sums back
        stage(ch, (ch - ch0) & 1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    ch = ch0;
    // Whether all of the part's chunks fit a digit pass's sums; if not, 15 do, whatever
    // their weights (a chunk's q0 is at most 64 * 2^16 / 2^6, its r1 64 * 32).
    int most = 15;
    if (passes > 1) {
        int sum0 = 0, sum1 = 0;
        for (int i = ch0 + lane; i < ch1; i += 64) {
            const Bounds u = bd[2 * i], v = bd[2 * i + 1];
            sum0 = min(sum0 + 17 * max(u.q0, v.q0), kLimit + 1);
            sum1 = min(sum1 + 271 * max(u.r1, v.r1), kLimit + 1);
        }
        for (int off = 32; off > 0; off >>= 1) {
            sum0 = min(sum0 + __shfl_xor(sum0, off), kLimit + 1);
            sum1 = min(sum1 + __shfl_xor(sum1, off), kLimit + 1);
        }
        if (__builtin_amdgcn_readfirstlane(max(sum0, sum1)) <= kLimit) most = ch1 - ch0;
    }
    static_assert(15 * 17 * 64 * 1024 <= kLimit && 15 * 271 * 64 * 32 <= kLimit, "15 chunks of a digit pass");
    for (int pass = 1; pass < passes;) {
        const int stop = min(ch1, ch + most);
        clear();
        // A chunk's two matrices are staged beside the parked sums during the chunk before,
        // its digits loaded kAhead chunks before: a pass touches them once, and what comes
        // from beyond L2 takes as long as several chunks. Where only some blocks have
        // digits of this pass, an entry of hmax for each pixel tells. (256 -> 256 channels
        // 3 x 3 on 14 x 14 at batch 128 over all of int32, four passes: 276 us with a
        // chunk's loads issued during the one before, 243 four ahead, 219 without a load
        // of the bounds between them, which waits for all that is on its way; with inputs
        // to 2^23, two passes, 166; one pass 135.)
        auto stage2 = [&](int c, int buf) {
            const uint32_t from = uint32_t(c) * uint32_t(kStageBytes) + uint32_t(fp6_lo(kP14, 0));
#pragma unroll
            for (int i = 0; i < kDigitStage / 1024; i += 4)
                if (i + wave < kDigitStage / 1024)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(
                        wr, (lds_ptr_t)(lds + kParked + buf * kDigitStage + (i + wave) * 1024), 16, uint32_t(lane * 16),
                        from + uint32_t(i + wave) * 1024u, 0, 0);
            asm volatile("" ::: "memory");   // the digits' loads come after it: it is waited for by count
        };
        auto run = [&](auto all_) {
            constexpr bool all = decltype(all_)::value;
            constexpr int kAhead = 4;
            auto fetch = [&](v8i &a0, v8i &a1, bool &some) {
                const uint32_t dbase = (uint32_t(cb) * 3u + uint32_t(pass - 1)) * uint32_t(p.NP) * 24u;
                bool in[2];
                v8i v[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int px = cb < CB ? pixel(t, r, s) : -1;
                    in[t] = px >= 0;
                    if constexpr (!all) in[t] = in[t] & (hmax[in[t] ? cb * p.nblk + (px >> 8) : 0] >= 252 + pass);
                    const v4i lo = __builtin_amdgcn_raw_buffer_load_b128(dr, in[t] ? dbase + uint32_t(px) * 16u : kOOB, 0, 0);
                    const v2i hi = __builtin_amdgcn_raw_buffer_load_b64(
                        dr, in[t] ? dbase + uint32_t(np16) + uint32_t(px) * 8u : kOOB, 0, 0);
                    v[t] = wide(lo, hi);
                }
                a0 = v[0];
                a1 = v[1];
                some = all || __ballot(in[0] | in[1]) != 0;
                step();
                if (!p.d.even) step();
            };
            v8i q[kAhead][2];
            bool some[kAhead];
            seek(ch);
            stage2(ch, 0);
#pragma unroll
            for (int u = 0; u < kAhead; ++u) fetch(q[u][0], q[u][1], some[u]);
            asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            int buf = 0;
            for (;;) {
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const v8i h[2] = {q[u][0], q[u][1]};
                    const bool now = some[u];
                    if (ch + 1 < ch1) stage2(ch + 1, buf ^ 1);
                    fetch(q[u][0], q[u][1], some[u]);
                    if (now) {
                        const unsigned char *st = lds + kParked + buf * kDigitStage - fp6_lo(kP14, 0);
#pragma unroll
                        for (int m = 0; m < 2; ++m) {
                            const int l8 = m ? lane8x : lane * 8;
                            const v8i a = wide(*reinterpret_cast<const v4i *>(st + fp6_lo(kP14, m) + lane * 16),
                                               *reinterpret_cast<const v2i *>(st + fp6_hi(kP14, m) + l8));
                            const v8i w = wide(*reinterpret_cast<const v4i *>(st + fp6_lo(kW, m) + lane * 16),
                                               *reinterpret_cast<const v2i *>(st + fp6_hi(kW, m) + l8));
#pragma unroll
                            for (int t = 0; t < 2; ++t) {
                                c0[m][t] = mms<kE3M2, kE2M3, kP4x>(a, h[t], c0[m][t], sc);
                                c1[m][t] = mms<kE3M2, kE2M3, kP2x, kP4x>(w, h[t], c1[m][t], sc);
                            }
                        }
                    }
                    // The next chunk's share has landed (only this chunk's four loads of digits
                    // came later), every wave's behind the barrier; this one's have been read.
                    asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    buf ^= 1;
                    ++ch;
                    if (ch == stop) return;
                }
            }
        };
        if (hleast >= 252 + pass) run(std::true_type());
        else run(std::false_type());
        park(true, 5 * pass);
        if (ch == ch1) {
            ++pass;
            ch = ch0;
        }
    }
    emit(more, true);
}

constexpr int64_t round256(int64_t v) { return (v + 255) & ~int64_t(255); }

}  // namespace

MfmaLayout mfma_layout(const ConvGeom &g, bool shared, int tasks)
{
    MfmaLayout l;
    l.sampled = !shared && g.r == 1 && g.s == 1 && g.ph == 0 && g.pw == 0 && g.oh <= (g.h - 1) / g.sh + 1 &&
                g.ow <= (g.w - 1) / g.sw + 1;
    // Few channels would leave most of a 32-channel block empty: the columns of a tap
    // row become channels instead, if that saves a third of the blocks or more.
    const int64_t plain = int64_t((g.c + kBlockK - 1) / kBlockK) * g.s;
    const int64_t folded = (int64_t(g.c) * g.s + kBlockK - 1) / kBlockK;
    l.US = !shared && !l.sampled && g.s > 1 && 3 * folded <= 2 * plain ? g.s : 1;
    l.PH = l.sampled ? g.oh : g.h;
    l.PW = l.sampled || l.US > 1 ? g.ow : g.w;
    const int64_t cb = (int64_t(g.c) * l.US + kBlockK - 1) / kBlockK, t = int64_t(g.r) * (l.US > 1 ? 1 : g.s);
    const int64_t np = int64_t(g.n) * l.PH * l.PW, nq = int64_t(g.n) * g.oh * g.ow;
    // Extents whose products below could not be formed are far past every limit; the
    // end of the last tile of kPix output pixels is formed in 32 bits.
    if (cb <= 0 || t <= 0 || nq <= 0 || cb > (1 << 24) || t > (1 << 24) || np > (int64_t(1) << 31) ||
        nq > (int64_t(1) << 31) - kPix)
        return l;
    const int64_t nchunks = (cb * t + 1) / 2;
    const int64_t tiles_p = (nq + kPix - 1) / kPix, tiles_k = (g.k + kRows - 1) / kRows;
    const int64_t nblk = (np + 255) / 256;
    // 32-bit buffer offsets (an address past 2^31 marks a position outside x), 32-bit
    // block counts, and rows and columns in 16 bits (the extents, a window's start up
    // to a padding before them, a tap up to a window after it).
    constexpr int64_t kMax = int64_t(1) << 31;
    l.fits = cb * np * kXpBytes < kMax - 512 && nchunks * kStageBytes < kMax - 65536 && tiles_p * tiles_k < kMax / 4 &&
             tiles_k * nchunks < kMax / 8 && cb * nblk < kMax / 4 && int64_t(g.n) * g.k * g.oh * g.ow < kMax &&
             std::max(l.PH, l.PW) < 16384 && std::max(g.r, g.s) < 8192 &&
             std::max(std::abs(g.ph), std::abs(g.pw)) < 8192;
    if (!l.fits) return l;
    l.CB = int(cb);
    l.even = l.CB % 2 == 0;
    l.xp_bytes = size_t(round256(cb * np * kXpBytes));
    l.dig_bytes = size_t(round256(cb * np * kDigBytes));
    l.hm_bytes = size_t(round256(cb * nblk));
    l.wa_bytes = size_t(tiles_k * nchunks * kStageBytes);
    l.bd_bytes = size_t(round256(2 * tiles_k * nchunks * int64_t(sizeof(Bounds))));
    l.NP = int(np);
    l.nblk = int(nblk);
    l.nchunks = int(nchunks);
    l.tiles_p = int(tiles_p);
    l.tiles_k = int(tiles_k);
    // Two workgroups fit a CU: a smaller grid splits the reduction, keeping two chunks
    // per part. That pays for long reductions only: y is filled first, its parts are
    // added to it and an epilogue is a pass of its own, while a workgroup alone on a CU
    // takes 2.2 us a chunk and two together 3.7. Measured (plans with a ReLU; without)
    // split and whole: 196 tiles of 18 chunks 62.5, 56.5 and 54.2, 54.8 us; 148 of 16
    // 63.6, 58.1 and 56.4, 55.7; 92 of 8 42.5, 36.6 and 33.3, 33.2; the other way 148 of
    // 18 55.9, 50.0 and 53.6, 54.5; 64 of 8 32.2, 28.0 and 30.6, 30.0; 200 of 72 148,
    // 144 and 158, 160.
    const int64_t tiles = tiles_p * tiles_k * tasks;
    int64_t splits = 1;
    if (tiles < 9 * nchunks) splits = std::max<int64_t>(1, std::min<int64_t>(512 / tiles, nchunks / 2));
    l.cps = int((nchunks + splits - 1) / splits);
    l.splits = int((nchunks + l.cps - 1) / l.cps);
    return l;
}

// The vector kernels keep the smallest problems, where a call is launches and
// latency: traced on MI355X, 40 -> 65 channels 3 x 3 on 9 x 9, batch 3 (0.6 M terms)
// takes 13.0 us there and 18.6 here, 512 -> 10 on 7 x 7, batch 32 (8 M, ten of the 64
// rows of a tile in use) 15.7 and 19.7; 64 -> 64 3 x 3 on 14 x 14 (7 M) 24.1 and
// 21.4, 128 -> 128 3 x 3 on 28 x 28 (116 M) 30.6 and 22.2, and 256 -> 256 3 x 3 on
// 14 x 14 at batch 128 (14.8 G) 935 and 150. From 50 M terms a few rows of a tile are
// enough (eager calls): 64 -> 1 3 x 3 on 56 x 56 at batch 32 (58 M) 198 and 46, 256 -> 4 on
// 28 x 28 at batch 8 (58 M) 68 and 27, 1024 -> 8 1 x 1 on 14 x 14 at batch 32 (51 M) 38 and
// 23. A LinearShift (256 rows or more here) takes five launches there: 128 -> 64 at batch
// 300 (2.5 M) 26.4 against 19.5.
bool mfma_prefer(const ConvGeom &g, int64_t terms)
{
    const bool linear = g.h == 1 && g.w == 1 && g.r == 1 && g.s == 1;
    return linear || (g.k > 16 && terms >= 4000000) || terms >= 50000000;
}

// By both paths' times (us, fitted to eager calls of 295 problems of 4 - 28 terms a row,
// 3 - 256 channels and 25 - 2097 thousand pixels, within 15 % of nearly all; the choice is
// 0.3 % off the best). On the matrix cores: x read and packed at 4 TB/s, whole tiles at 139
// T terms/s, each row's sums at 6.6 T/s and y at 9.2 TB/s. On the vector kernels: y at 3.7
// TB/s, or a third of that and 11.5 T terms/s of at least 32 rows; an input gradient
// re-packs its codes first (4). Measured there and on the matrix cores: 4 -> 24 1 x 1 on 112
// x 112 at batch 8 14 and 20, 8 -> 64 on 56 x 56 at batch 64 26 and 39, 1 -> 64 3 x 3 29 and
// 45, 3 -> 24 34 and 44, 3 -> 64 104 and 75 (512 x 512, batch 2), 16 -> 128 1 x 1 55 and 49
// (56 x 56, batch 64); gradients of 64 -> 4 1 x 1 on 512 x 512 at batch 8 207 and 226, 64 -> 16
// on 112 x 112 28 and 22.
bool mfma_padded(const ConvGeom &g, const MfmaLayout &l, bool gradient)
{
    const bool linear = g.h == 1 && g.w == 1 && g.r == 1 && g.s == 1;
    if (linear || double(g.crs) >= 0.45 * 64.0 * l.nchunks || g.r > 5 || g.s > 5) return false;
    const double x = 4.0 * g.n * double(g.c) * g.h * g.w, nq = double(g.n) * g.oh * g.ow, y = 4.0 * nq * g.k;
    const double rows = double(l.tiles_k) * kRows;
    const double matrix = 13.0 + (x + double(kXpBytes) * l.CB * l.NP) / 4.0e6 +
                          double(l.tiles_p) * kPix * rows * l.nchunks * 64.0 / 139e6 + nq * rows / 6.6e6 + y / 9.2e6;
    const double issue = nq * std::max(32, (g.k + 15) / 16 * 16) * g.crs / 11.5e6;
    const double vector = 12.0 + (gradient ? 4.0 : 1.0) + std::max(y / 3.7e6, issue + y / 11.5e6);
    return vector <= matrix;
}

// In microseconds on MI355X (graph replays): two launches and what a tile does
// besides its products (10), the packed copy of x written and read at 5.5 TB/s, the
// products of whole tiles at 130 T terms/s (2.2 a chunk at least), y at 4 TB/s, 15 for
// a split reduction. Measured (estimated): 256 -> 256 3x3 on 14x14 at batch 128 138
// (138), 64 -> 64 3x3 on 56x56 177 (181), 1024 -> 256 on 14x14 95 (98), 512 -> 512 3x3
// on 7x7 at batch 32 63 (55), 4096 -> 4096 at batch 256 64 (60), 512 -> 128 on 28x28
// 135 (136), 64 -> 256 on 56x56 196 (195), the 7x7 stem 376 (355), 128 -> 128 3x3 on
// 28x28 at batch 8 32 (35).
double mfma_plan_us(const MfmaTask *tasks, size_t ntasks, int64_t x_elems)
{
    const MfmaLayout &l = tasks[0].l;
    double us = 10.0 + (4.0 * x_elems + 2.75 * 32.0 * l.CB * l.NP) / 5.5e6;
    bool split = false;
    for (size_t i = 0; i < ntasks; ++i) {
        const MfmaTask &t = tasks[i];
        us += std::max(double(t.l.tiles_p) * kPix * t.l.tiles_k * kRows * t.l.nchunks * 64.0 / 130e6,
                       ntasks == 1 ? 2.2 * t.l.cps : 0.0) +
              4.0 * t.g.n * double(t.g.k) * t.g.oh * t.g.ow / 4e6;
        split = split || t.l.splits > 1;
    }
    if (split) us += 15.0;
    return us;
}

MfmaWeights mfma_forward_weights(const ConvGeom &g)
{
    MfmaWeights w;
    w.R = g.r;
    w.S = g.s;
    w.wpr = int(row_words_bits(g.crs, g.bits));
    w.bits = g.bits;
    return w;
}

MfmaWeights mfma_phase_weights(const ConvGeom &f, const GradPhase &ph)
{
    MfmaWeights w;
    w.R = f.r;
    w.S = f.s;
    w.r0 = ph.r0 + f.sh * (ph.g.r - 1);   // the phase's taps in reverse order
    w.dr = -f.sh;
    w.s0 = ph.s0 + f.sw * (ph.g.s - 1);
    w.ds = -f.sw;
    w.adjoint = true;
    w.wpr = int(row_words_bits(f.crs, f.bits));
    w.bits = f.bits;
    return w;
}

namespace {

Reduction reduction(const MfmaTask &t)
{
    Reduction d{};
    d.CB = t.l.CB;
    d.R = t.g.r;
    d.S = t.l.US > 1 ? 1 : t.g.s;
    d.US = t.l.US;
    d.C = t.g.c * t.l.US;
    d.even = t.l.even;
    d.nchunks = t.l.nchunks;
    return d;
}

OutMap full_output(const MfmaTask &t)
{
    const ConvGeom &g = t.g;
    return t.map.dense() ? OutMap{0, g.k * g.oh * g.ow, g.oh * g.ow, g.ow, 1} : t.map;
}

}  // namespace

hipError_t mfma_prepare(const MfmaTask *tasks, int ntasks, const void *x, int act_bytes, const uint32_t *wp,
                        unsigned char *input, const int32_t *bias, int32_t *y, hipStream_t st)
{
    if (ntasks < 1 || ntasks > kMfmaTasks) return hipErrorInvalidValue;
    PrepArgs a{};
    a.x = x;
    a.wp = wp;
    if (x) {
        const MfmaTask &t = tasks[0];
        const ConvGeom &g = t.g;
        const MfmaLayout &l = t.l;
        a.xp = input;
        a.dig = input + l.xp_bytes;
        a.hmax = a.dig + l.dig_bytes;
        PackParams &k = a.p;
        k.C = g.c; k.W = g.w; k.HW = g.h * g.w;
        k.NP = l.NP; k.PHW = l.PH * l.PW;
        k.sh = l.sampled ? g.sh : 1;
        k.sw = l.sampled || l.US > 1 ? g.sw : 1;
        k.pw = l.US > 1 ? g.pw : 0;
        k.US = l.US;
        k.nblk = l.nblk;
        k.div_phw = make_fastdiv(uint32_t(k.PHW));
        k.div_pw = make_fastdiv(uint32_t(l.PW));
        k.div_us = make_fastdiv(uint32_t(l.US));
        a.pblocks = l.CB * l.nblk;
    }
    int64_t fills = 0;
    for (int i = 0; i < ntasks; ++i) {
        const MfmaTask &t = tasks[i];
        const ConvGeom &g = t.g;
        if (!t.l.fits) return hipErrorInvalidValue;
        if (wp) {
            WeightTask &w = a.w[i];
            w.d = reduction(t);
            w.w = t.w;
            w.fmt = code_fmt(t.w.bits);
            w.K = g.k;
            w.blocks = 2 * t.l.tiles_k * t.l.nchunks;
            w.wa = t.weights;
            w.bounds = reinterpret_cast<Bounds *>(t.weights + t.l.wa_bytes);
            a.wblocks += w.blocks;
        }
        FillParams &f = a.f[i];
        if (t.l.splits > 1 && y) {
            const OutMap m = full_output(t);
            f.y = y;
            f.bias = bias;
            f.K = g.k; f.OHOW = g.oh * g.ow; f.OW = g.ow; f.NK = g.n * g.k;
            f.ybase = int(m.base); f.ynst = m.nstride; f.ykst = m.kstride; f.yrst = m.rstride; f.ycst = m.cstride;
            f.div_ohow = make_fastdiv(uint32_t(f.OHOW));
            f.div_ow = make_fastdiv(uint32_t(f.OW));
            f.div_k = make_fastdiv(uint32_t(f.K));
            f.blocks = int(std::min<int64_t>((int64_t(f.NK) * f.OHOW + 1023) / 1024, 2048));
            fills += f.blocks;
        }
    }
    const int64_t blocks = int64_t(a.wblocks) + a.pblocks + fills;
    if (blocks == 0) return hipSuccess;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid{unsigned(blocks)}, block{256u};
    if (act_bytes == 2) hipLaunchKernelGGL(mfma_prep_kernel<int16_t>, grid, block, 0, st, a);
    else if (act_bytes == 1) hipLaunchKernelGGL(mfma_prep_kernel<int8_t>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(mfma_prep_kernel<int32_t>, grid, block, 0, st, a);
    return hipGetLastError();
}

hipError_t mfma_multiply(const MfmaTask *tasks, int ntasks, const unsigned char *input, const int32_t *bias,
                         int32_t *y, const Epilogue &epi, hipStream_t st)
{
    if (ntasks < 1 || ntasks > kMfmaTasks) return hipErrorInvalidValue;
    ProductArgs a{};
    a.xp = input;
    a.dig = input + tasks[0].l.xp_bytes;
    a.hmax = a.dig + tasks[0].l.dig_bytes;
    a.bias = bias;
    a.y = y;
    a.epi = epi;
    int64_t tiles = 0;
    int splits = 1;
    for (int i = 0; i < ntasks; ++i) {
        const MfmaTask &t = tasks[i];
        const ConvGeom &g = t.g;
        const MfmaLayout &l = t.l;
        if (!l.fits) return hipErrorInvalidValue;
        MfmaParams &p = a.p[i];
        p.d = reduction(t);
        p.PH = l.PH; p.PW = l.PW; p.PHW = l.PH * l.PW; p.NP = l.NP;
        p.sh = l.sampled ? 1 : g.sh;
        p.sw = l.sampled || l.US > 1 ? 1 : g.sw;
        p.ph = g.ph;
        p.pw = l.US > 1 ? 0 : g.pw;
        p.K = g.k; p.OHOW = g.oh * g.ow; p.NQ = int(int64_t(g.n) * p.OHOW);
        p.tiles_p = l.tiles_p; p.tiles_k = l.tiles_k; p.cps = l.cps; p.nblk = l.nblk;
        p.atomic_out = l.splits > 1;
        p.fuse_epi = epi.any() && l.splits == 1;
        const OutMap m = full_output(t);
        p.ybase = int(m.base); p.ynst = m.nstride; p.ykst = m.kstride; p.yrst = m.rstride; p.ycst = m.cstride;
        p.rowmajor = m.kstride == 1 && p.OHOW == 1;
        p.xp_bytes = uint32_t(l.xp_bytes);
        p.div_ohow = make_fastdiv(uint32_t(p.OHOW));
        p.div_ow = make_fastdiv(uint32_t(g.ow));
        p.wa = t.weights;
        p.bounds = reinterpret_cast<const Bounds *>(t.weights + l.wa_bytes);
        tiles = std::max(tiles, int64_t(l.tiles_p) * l.tiles_k);
        splits = std::max(splits, l.splits);
    }
    hipLaunchKernelGGL(mfma_conv_kernel, dim3(unsigned((tiles + 7) / 8 * 8), unsigned(splits), unsigned(ntasks)),
                       dim3(256), 0, st, a);
    hipError_t e = hipGetLastError();
    // The epilogue of a split task (one on its own, dense) is a pass over y.
    if (e == hipSuccess && epi.any() && tasks[0].l.splits > 1) e = run_epilogue(tasks[0].g, y, epi, st);
    return e;
}

}  // namespace ds
