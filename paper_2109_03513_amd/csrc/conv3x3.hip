// Direct 3x3 / pad-1 convolution, stride 1 or 2, over ESB codes on the fp8 MFMA
// of gfx950 (Sec. 4.2: the convolution stage; products of codes by eq. (15),
// exact as in the implicit-GEMM path), for input and output channels that are
// multiples of 64.
//
// The implicit-GEMM kernels fetch and decode every input element once per
// filter tap it meets, nine times for a 3x3 filter.  Here a workgroup owns TM
// consecutive output pixels (flattened over the batch) and 64 output channels,
// and runs over the input channels in chunks of 64:
//  * per chunk, the input rows under the tile are decoded to E4M3 once into an
//    LDS patch, one 64-byte row per input pixel.  Every image is seen with a
//    zero row above and below it and a zero column left and right (the
//    padding), so a tile may cross images: output pixel (n, p, q) and tap
//    (r, s) read padded row n (H + 2) + st p + r - R0 (R0 the first padded row of
//    the tile) and padded column st q + s.  With stride 2 a patch row holds the
//    even padded columns first, then the odd ones, so that a tap over 32
//    consecutive output pixels still reads consecutive patch pixels.  The four 16-byte chunks of a patch pixel are
//    stored in the order chunk ^ ((pixel / 4) % 4), so that 16 consecutive
//    pixels read at one chunk (a quarter-wave of a fragment load) hit 16
//    different bank groups;
//  * per chunk the filter slice (64 outputs x 9 taps x 64 channels) is decoded
//    into LDS; with one chunk (64 input channels) it is decoded once per
//    workgroup and stays (workgroups are persistent over their tiles);
//  * the codes of the next chunk (or tile) are loaded into registers while the
//    current chunk's MFMAs run;
//  * per tap one v_mfma_scale_f32_32x32x64_f8f6f4 per 32 x 32 block;
//  * the epilogue is the contraction's: acc = the fp32 sum times 2^shift
//    (an exact integer), y0 = fl32(s fl32(acc)) and the fused post-processing.
//    fp32 outputs alone and codes alone, without the affine step, leave straight
//    from the accumulators (store_direct) where the kernel has an instance for
//    them; every other form makes a round trip through LDS, four consecutive
//    channels per lane.
// The fp32 sums are exact under the same admission rule as the implicit-GEMM
// fp8 path (every product at most 2^12, 9 C x the largest product < 2^24), so
// the results equal that path's bit for bit.
#include "esb_internal.h"

namespace esb {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;           // four waves
constexpr int NT = 64;                  // output channels per workgroup
constexpr int CK = 64;                  // input channels per chunk
constexpr int TAPS = 9;
constexpr int WST = TAPS * CK + 16;     // LDS bytes per output channel of the filter slice:
                                        // 148 dwords, so the 16 lanes of a quarter-wave
                                        // (16 channels) take 16 different bank groups
constexpr int kPatchMax = 40 * 1024;    // bytes of the input patch
constexpr int kMaxCols = kThreads / 4;  // Q + 2: one thread per 16-byte chunk of a patch row
constexpr int SLAB = 72;                // fp32 row stride of the epilogue slabs
constexpr int kMaxFill = 10;            // patch chunks per thread and chunk of channels
constexpr int kFewFill = 5;             // the same where this many suffice
constexpr int kMidFill = 9;             // likewise (several chunks, 128-pixel tiles), and
constexpr int kSumsFill = 8;            // with int32 sums: each one more spills there
constexpr int kWPer = NT * TAPS * 4 / kThreads;   // filter chunks per thread (9)
static_assert(4 * 32 * SLAB * 4 <= kPatchMax, "epilogue slabs fit the patch");
static_assert(kWPer * kThreads == NT * TAPS * 4, "whole filter chunks per thread");
constexpr int64_t kMultiMaxPixels = 16384;   // several chunks: at most this many output pixels

struct Conv3Params {
    const uint8_t* x;          // [N, H, W, C] codes (H = P, W = Q)
    const uint8_t* w;          // [K, 3, 3, C] codes
    const float* alphaX;
    const float* alphaW;
    int32_t* acc;              // [M, K] or NULL
    float* y;                  // [M, K] or NULL
    MmaDecode dx, dw;
    Post post;
    int N, P, Q, M;            // M = N P Q output pixels
    int H, W, st;              // input height and width, stride (1, or 2 in k_conv3x3)
    int half;                  // stride 2: padded columns of even index, (W + 3) / 2
    int C, K;                  // channels in and out (multiples of 64)
    int ntm, ntn;              // pixel tiles, channel tiles
    int out_shift;             // acc = fl32 sum * 2^out_shift
    int kX, kW;
    int direct;                // outputs straight from the registers: 1 fp32, 2 codes, 0 neither
};

__device__ __forceinline__ uint4 dec16(uint4 v, const MmaDecode& d) {
    return make_uint4(dec_f8(v.x, d), dec_f8(v.y, d), dec_f8(v.z, d), dec_f8(v.w, d));
}

// LDS byte offset of chunk c (0..3) of patch pixel pix.
__device__ __forceinline__ int patch_off(int pix, int c) {
    return (pix << 6) | ((c ^ ((pix >> 2) & 3)) << 4);
}

// One 32 x 32 block of accumulators into a slab of rows (pixels) of sl floats at column c0:
// register 4 g + e is pixel lane % 32, channel 8 g + 4 (lane / 32) + e.
__device__ __forceinline__ void to_slab(float* slab, int sl, const v16f& a, int c0, int lane, float s,
                                        int shift) {
#pragma unroll
    for (int g = 0; g < 4; g++) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; e++) v[e] = s * ldexpf(a[4 * g + e], shift);
        *(f32x4*)(slab + (lane & 31) * sl + c0 + 8 * g + 4 * (lane >> 5)) = v;
    }
}
__device__ __forceinline__ void to_slab_int(float* slab, int sl, const v16f& a, int c0, int lane,
                                            int shift) {
#pragma unroll
    for (int g = 0; g < 4; g++) {
        v4i v;
#pragma unroll
        for (int e = 0; e < 4; e++) v[e] = (int32_t)ldexpf(a[4 * g + e], shift);
        *(v4i*)(slab + (lane & 31) * sl + c0 + 8 * g + 4 * (lane >> 5)) = v;
    }
}

// The outputs of one 32-pixel block from a wave's slab (row stride sl floats,
// WCOLS channels from channel c0): four consecutive channels per lane.  AHEAD:
// the residual loads four at a time in flight before they are used (for kernels
// with one block per wave: with two, the registers do not fit); else one output
// group after the other.  Returns the lane's max |z| bit pattern.
template <int WCOLS, bool AHEAD>
__device__ __forceinline__ uint32_t store_block(const Conv3Params& p, const float* slab, int sl,
                                                int mrow, int c0, int lane, float qa) {
    constexpr int NIT = 32 * WCOLS / 256;
    uint32_t amax = 0;
    // Post-processing without a per-channel affine and without codes (ReLU /
    // residual / max|z| only) takes lean code instead of the general
    // post-processing; the unrolled form also takes the plain output (the rolled
    // form keeps its own plain loop, which issues no global load between the
    // stores).  z = v + 0 is the affine step of the general path with a = 1, b = 0
    // (one rounding: it turns -0 into +0), so both agree bit for bit.
    const bool lean = p.post.on ? (!p.post.a && !p.post.b && !p.post.codes) : AHEAD;
    const bool on = p.post.on != 0;
    const float* res = on ? p.post.res : nullptr;
    const bool relu = on && p.post.relu;
    const bool am = on && p.post.absmax;
    auto lean4 = [&](int64_t o, f32x4 z, f32x4 r) {
        if (on) {
#pragma unroll
            for (int c = 0; c < 4; c++) z[c] = z[c] + 0.0f;
        }
        if (res) {
#pragma unroll
            for (int c = 0; c < 4; c++) z[c] = z[c] + r[c];
        }
        if (relu) {
#pragma unroll
            for (int c = 0; c < 4; c++) z[c] = z[c] > 0.0f ? z[c] : 0.0f;
        }
        if (p.y) {
            float* d = p.y + o;
            if (((uintptr_t)d & 15) == 0) {
                *(f32x4*)d = z;
            } else {
#pragma unroll
                for (int c = 0; c < 4; c++) d[c] = z[c];
            }
        }
        uint32_t mz = 0;
        if (am) {
#pragma unroll
            for (int c = 0; c < 4; c++) mz = max(mz, __float_as_uint(z[c]) & 0x7fffffffu);
        }
        return mz;
    };
    auto res4 = [&](int64_t o) {
        f32x4 r = {0.0f, 0.0f, 0.0f, 0.0f};
        if (res) {
            const float* q = res + o;
            if (((uintptr_t)q & 15) == 0) {
                r = *(const f32x4*)q;
            } else {
#pragma unroll
                for (int c = 0; c < 4; c++) r[c] = q[c];
            }
        }
        return r;
    };
    if (AHEAD && lean) {   // unrolled, the residual loads four at a time ahead of use
#pragma unroll
        for (int k0 = 0; k0 < NIT; k0 += 4) {
            f32x4 rr[4];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int e = 4 * lane + 256 * (k0 + k), row = e / WCOLS, col = e - row * WCOLS;
                const int m = mrow + row;
                rr[k] = (k0 + k < NIT && m < p.M) ? res4((int64_t)m * p.K + c0 + col)
                                                  : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            }
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int e = 4 * lane + 256 * (k0 + k), row = e / WCOLS, col = e - row * WCOLS;
                const int m = mrow + row;
                if (k0 + k < NIT && m < p.M) {
                    const int64_t o = (int64_t)m * p.K + c0 + col;
                    const f32x4 v = *(const f32x4*)(slab + row * sl + col);
                    amax = max(amax, lean4(o, v, rr[k]));
                }
            }
        }
        return amax;
    }
    if (!AHEAD) {
#pragma unroll 1
        for (int e = 4 * lane; e < 32 * WCOLS; e += 256) {
            const int row = e / WCOLS, col = e - row * WCOLS;
            const int m = mrow + row;
            if (m < p.M) {
                const int ch = c0 + col;
                const int64_t o = (int64_t)m * p.K + ch;
                const f32x4 v = *(const f32x4*)(slab + row * sl + col);
                if (lean) {
                    amax = max(amax, lean4(o, v, res4(o)));
                } else if (p.post.on) {
                    amax = max(amax, post_store4(p.post, p.y, o, ch, v, 4, qa));
                } else if (p.y) {
                    if (((uintptr_t)(p.y + o) & 15) == 0) {
                        *(f32x4*)(p.y + o) = v;
                    } else {
#pragma unroll
                        for (int c = 0; c < 4; c++) p.y[o + c] = v[c];
                    }
                }
            }
        }
        return amax;
    }
    if (p.post.on) {
#pragma unroll
        for (int k0 = 0; k0 < NIT; k0 += 4) {   // four residual loads in flight at a time
            f32x4 rr[4];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int e = 4 * lane + 256 * (k0 + k), row = e / WCOLS, col = e - row * WCOLS;
                const int m = mrow + row;
                rr[k] = (k0 + k < NIT && m < p.M) ? post_res4(p.post, (int64_t)m * p.K + c0 + col)
                                                  : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            }
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int e = 4 * lane + 256 * (k0 + k), row = e / WCOLS, col = e - row * WCOLS;
                const int m = mrow + row;
                if (k0 + k < NIT && m < p.M) {
                    const int ch = c0 + col;
                    const f32x4 v = *(const f32x4*)(slab + row * sl + col);
                    amax = max(amax, post_apply4(p.post, p.y, (int64_t)m * p.K + ch, ch, v, rr[k], qa));
                }
            }
        }
    } else if (p.y) {
#pragma unroll
        for (int k = 0; k < NIT; k++) {
            const int e = 4 * lane + 256 * k, row = e / WCOLS, col = e - row * WCOLS;
            const int m = mrow + row;
            if (m < p.M) {
                const int64_t o = (int64_t)m * p.K + c0 + col;
                const f32x4 v = *(const f32x4*)(slab + row * sl + col);
                if (((uintptr_t)(p.y + o) & 15) == 0) {
                    *(f32x4*)(p.y + o) = v;
                } else {
#pragma unroll
                    for (int c = 0; c < 4; c++) p.y[o + c] = v[c];
                }
            }
        }
    }
    return amax;
}

// The outputs of one 32-pixel block (pixels mrow + lr) and NB blocks of 32 channels from c0
// straight from the accumulators: the filter is the first matrix operand, so register
// 4 g + e of block j is channel c0 + 32 j + 8 g + 4 lg + e, four consecutive channels per four
// registers.  fp32 outputs (with a residual already in res, ReLU, max|z|) leave in 16-byte
// stores; codes, after two swaps of lane halves, 16 per lane.  Against the trip through LDS
// slabs this saves 2 x 128 bytes of LDS traffic per pixel and channel block and every barrier
// of the epilogue (batch 64, codes out: 256 channels
// at 14 x 14 21.5 -> 18.0 us, 128 at 28 x 28 32.0 -> 26.3; fp32 out: 128 at 28 x 28 23.2 -> 20.7,
// 512 at 7 x 7 21.8 -> 20.6).  z = v + 0 is the affine step with a = 1, b = 0.
template <int NB>
__device__ __forceinline__ void load_res(const Conv3Params& p, f32x4 (&res)[4 * NB], int mrow, int c0,
                                         int lane) {
    const int m = min(mrow + (lane & 31), p.M - 1);
    const float* r = p.post.res + (int64_t)m * p.K + c0 + 4 * (lane >> 5);
#pragma unroll
    for (int q = 0; q < 4 * NB; q++) res[q] = *(const f32x4*)(r + 8 * q);
}

template <int NB, int OUT>
__device__ __forceinline__ uint32_t store_direct(const Conv3Params& p, const v16f (&a)[NB],
                                                 const f32x4 (&res)[4 * NB], int mrow, int c0, int lane,
                                                 float s, float qa) {
    const int m = mrow + (lane & 31), lg = lane >> 5;
    const bool in = m < p.M;
    const bool on = p.post.on != 0, relu = p.post.relu != 0;
    const bool has_res = OUT == 1 && p.post.res != nullptr;
    uint32_t amax = 0;
    auto value = [&](int j, int g) {
        f32x4 z;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            z[e] = s * ldexpf(a[j][4 * g + e], p.out_shift);
            if (on) z[e] = z[e] + 0.0f;
            if (has_res) z[e] = z[e] + res[4 * j + g][e];
            if (relu) z[e] = z[e] > 0.0f ? z[e] : 0.0f;
            amax = max(amax, __float_as_uint(z[e]) & 0x7fffffffu);
        }
        return z;
    };
    if (OUT == 1) {
        float* y = p.y + (int64_t)m * p.K + c0 + 4 * lg;
#pragma unroll
        for (int j = 0; j < NB; j++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const f32x4 z = value(j, g);
                if (in) *(f32x4*)(y + 32 * j + 8 * g) = z;
                __builtin_amdgcn_sched_barrier(0);   // four outputs at a time: registers
            }
    } else {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        const bool ok = alpha_valid(qa), fast = fast_scale(qa);
        const float r = 1.0f / qa;
        uint8_t* o = p.post.codes + (int64_t)m * p.K + c0 + 16 * lg;
#pragma unroll
        for (int j = 0; j < NB; j++) {
            uint32_t c[4];
#pragma unroll
            for (int g = 0; g < 4; g++)
                c[g] = ok ? code4(value(j, g), qa, r, fast, p.post.pp) : p.post.pp.zero_code * 0x01010101u;
            const u32x2 s02 = __builtin_amdgcn_permlane32_swap(c[0], c[2], false, false);
            const u32x2 s13 = __builtin_amdgcn_permlane32_swap(c[1], c[3], false, false);
            if (in) *(uint4*)(o + 32 * j) = make_uint4(s02[0], s02[1], s13[0], s13[1]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    return in ? amax : 0u;
}

// Two waves per SIMD: two workgroups share a CU (LDS 2 x 78 KB).  TMB: 32-pixel
// blocks per tile (8, 4 or 2; four waves take TMB x 2 blocks of 32 x 32).
// MULTI: more than one chunk of input channels (the filter slices then travel
// per chunk; at most 4 blocks per tile, for the registers).  ACC: the int32
// sums are written too (a separate instance: keeping both outputs live costs
// registers).  KG == 2: one workgroup of eight waves per CU, whose two halves take every
// other chunk of input channels, each with its own patch and filter slice, and add their
// (exact) sums at the end: where there are no more tiles than CUs, a second workgroup would
// find no tile, and four waves alone leave fill, barriers and LDS reads uncovered
// (512 -> 512 at 7 x 7, batch 64, 200 tiles: fp32 out 23.4 us with KG 1, 20.7 with 2; codes
// 22.4 and 20.0; all outputs 29.8 and 25.1.  Six chunks, 384 -> 384 at 14 x 14, batch 16: 17.4
// and 16.0.  Four chunks gain too little for instances of their own: 256 -> 256 at 14 x 14,
// batch 16, codes 12.1 and 12.1, fp32 out 11.7 and 11.4).
// FILL: patch chunks per thread, at least patch rows / rows per step; the unused ones of a
// larger FILL cost registers, repeated loads of one place and decoding.
template <int TMB, bool MULTI, int OUT, int FILL, int KG = 1>
__global__ __launch_bounds__(kThreads * KG) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_conv3x3(Conv3Params p) {
    constexpr int TM = 32 * TMB;
    constexpr int NMB = TMB >= 8 ? 2 : 1;    // output blocks of a wave: NMB x NNB
    constexpr int NNB = TMB >= 4 ? 2 : 1;
    static_assert(4 * NMB * NNB == 2 * TMB, "four waves cover the tile");
    static_assert(!MULTI || TMB <= 4, "several chunks: at most 4 pixel blocks");
    constexpr bool ACC = OUT == 3;
    static_assert(KG == 1 || (MULTI && !ACC), "halves of the reduction: several chunks");
    __shared__ __align__(16) uint8_t wlds_all[KG][NT * WST];
    __shared__ __align__(16) uint8_t patch_all[KG][kPatchMax];
    const int lane = threadIdx.x & 63;
    const int half = KG == 2 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads) : 0;
    const int tid = (int)threadIdx.x - half * kThreads;   // within the half
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint8_t* const wlds = wlds_all[half];
    uint8_t* const patch = patch_all[half];
    const int lr = lane & 31, lg = lane >> 5;
    // this wave's blocks: pixel blocks mbw + i (i < NMB), channel blocks nbw + j (j < NNB)
    const int mbw = TMB == 8 ? 2 * wave : (TMB == 4 ? wave : wave >> 1);
    const int nbw = TMB == 2 ? (wave & 1) : 0;

    const int nt = (int)blockIdx.x % p.ntn;          // this workgroup's output channels
    const int n0 = nt * NT;
    const int wg = (int)blockIdx.x / p.ntn, nwg = (int)gridDim.x / p.ntn;
    const int nchunks = MULTI ? p.C / CK : 1;

    float s = 0.0f;   // int32 sums alone: the scales may be NULL
    if (!ACC || p.y || p.post.on) s = ldexpf(p.alphaX[0] * p.alphaW[0], -(p.kX + p.kW));
    const float qa = post_alpha(p.post);
    uint32_t amax = 0;
    const int st = p.st;
    const int cols = p.W + 2, PP2 = p.H + 2, PQ = p.P * p.Q;
    // patch fill: thread t takes chunk t % (4 cols) of rows t / (4 cols), + rstep, ...
    const int cpr = 4 * cols;
    const int fci = tid % cpr, fri = tid / cpr, rstep = kThreads / cpr;
    const int fcol = fci >> 2, fc = fci & 3, iw = fcol - 1;
    const bool col_in = (unsigned)iw < (unsigned)p.W;
    // where padded column fcol sits in a patch row: stride 1 in order; stride 2 the
    // even columns first, then the odd ones, so that the taps of consecutive output
    // pixels (columns 2q + s) read consecutive patch pixels
    const int dcol = st == 1 ? fcol : ((fcol & 1) ? p.half + (fcol >> 1) : (fcol >> 1));
    const int tcol1 = st == 1 ? 1 : p.half, tcol2 = st == 1 ? 2 : 1;   // taps s = 1, 2
    // B fragments: channel 32 j + lr, bytes 32 lg .. + 31 of tap t
    const int boff = lr * WST + 32 * lg;
    const int64_t wrow = (int64_t)TAPS * p.C;        // filter bytes per output channel

    // The patch rows of a tile: padded rows R0 .. R0 + nrows - 1.
    auto rows_of = [&](int tile, int& R0, int& nrows) {
        const int m0 = tile * TM;
        const int i0 = m0 / PQ, p0 = (m0 - i0 * PQ) / p.Q;
        R0 = i0 * PP2 + st * p0;
        const int m1 = min(m0 + TM, p.M) - 1;
        const int i1 = m1 / PQ, p1 = (m1 - i1 * PQ) / p.Q;
        nrows = i1 * PP2 + st * p1 + 3 - R0;
    };
    // This thread's patch chunks of a tile (chunk u is row fri + u rstep): their places in the
    // input, and in bit u of vmask whether inside it (frows: the tile's patch rows; chunks
    // outside the input or past the rows load the input's first bytes, unused).
    uint4 raw[FILL], wraw[kWPer];
    uint32_t poff[FILL], vmask = 0;
    int frows = 0;
    auto prepare = [&](int tile) {
        int R0;
        rows_of(tile, R0, frows);
        const int pr = R0 + fri;
        int n = pr / PP2, hp = pr - n * PP2;             // padded row hp of image n
        vmask = 0;
#pragma unroll
        for (int u = 0; u < FILL; u++) {
            const int ih = hp - 1;
            const bool ok = fri < rstep && fri + u * rstep < frows && col_in && n < p.N &&
                            (unsigned)ih < (unsigned)p.H;
            poff[u] = (ok ? ((uint32_t)(n * p.H + ih) * p.W + iw) * (uint32_t)p.C : 0u) + 16 * fc;
            vmask |= ok ? (1u << u) : 0u;
            hp += rstep;
            while (hp >= PP2) { hp -= PP2; n++; }
        }
    };
    // The codes of one chunk of channels of the prepared tile and, with several chunks, this
    // thread's filter chunks (channel tid / 4, 16 bytes of every tap); every load in flight
    // at once.
    const uint8_t* const wthr = p.w + (n0 + (tid >> 2)) * wrow + 16 * (tid & 3);
    uint8_t* const wst = wlds + (tid >> 2) * WST + 16 * (tid & 3);
    auto fetch = [&](int ch) {
        const uint8_t* xc = p.x + CK * ch;
#pragma unroll
        for (int u = 0; u < FILL; u++) {
            raw[u] = *(const uint4*)(xc + poff[u]);
        }
        if (MULTI) {
#pragma unroll
            for (int u = 0; u < kWPer; u++) wraw[u] = *(const uint4*)(wthr + u * p.C + CK * ch);
        }
    };
    auto store_filter = [&]() {
#pragma unroll
        for (int u = 0; u < kWPer; u++) *(uint4*)(wst + 64 * u) = dec16(wraw[u], p.dw);
    };

    // ---- one chunk of channels: the filter once per workgroup, already in LDS
    if (!MULTI) {
#pragma unroll
        for (int u = 0; u < kWPer; u++) {   // rows of 576 contiguous bytes
            const int it = tid + u * kThreads, k = it / (TAPS * 4), rem = it - k * (TAPS * 4);
            wraw[u] = *(const uint4*)(p.w + (n0 + k) * wrow + 16 * rem);
        }
#pragma unroll
        for (int u = 0; u < kWPer; u++) {
            const int it = tid + u * kThreads, k = it / (TAPS * 4), rem = it - k * (TAPS * 4);
            *(uint4*)&wlds[k * WST + 16 * rem] = dec16(wraw[u], p.dw);
        }
    }
    if (wg < p.ntm && half < nchunks) {
        prepare(wg);
        fetch(half);
    }

    for (int tile = wg; tile < p.ntm; tile += nwg) {
        const int m0 = tile * TM;
        int R0, nrows;
        rows_of(tile, R0, nrows);

        // ---- per lane and output block: the patch pixel of tap (0, 0)
        int pb[NMB];
#pragma unroll
        for (int i = 0; i < NMB; i++) {
            const int m = min(m0 + 32 * (mbw + i) + lr, p.M - 1);   // rows past M: any pixel
            const int n = m / PQ, rem = m - n * PQ;
            const int pp = rem / p.Q, q = rem - pp * p.Q;
            pb[i] = (n * PP2 + st * pp - R0) * cols + q;
        }
        // one chunk: the filter fragments are the same for every tile, and the compiler would
        // move all nine taps of them into registers (144, spilled); an offset it cannot see
        // through keeps their reads here
        int btile = boff;
        if (!MULTI) asm volatile("" : "+v"(btile));
        v16f acc[NMB][NNB];
#pragma unroll
        for (int i = 0; i < NMB; i++)
#pragma unroll
            for (int j = 0; j < NNB; j++)
#pragma unroll
                for (int r = 0; r < 16; r++) acc[i][j][r] = 0.0f;

        for (int c0 = 0; c0 < nchunks; c0 += KG) {
            const int ch = c0 + half;
            const bool active = KG == 1 || ch < nchunks;   // the last chunk of an odd number
            __syncthreads();   // the previous chunk's (or tile's) reads of the LDS are done
            if (active && fri < rstep) {
#pragma unroll
                for (int u = 0; u < FILL; u++) {
                    const int i = fri + u * rstep;
                    if (i < frows) {
                        const uint4 v = ((vmask >> u) & 1u) ? dec16(raw[u], p.dx)
                                                            : make_uint4(0u, 0u, 0u, 0u);   // E4M3 +0
                        *(uint4*)&patch[patch_off(i * cols + dcol, fc)] = v;
                    }
                }
            }
            if (MULTI && active) store_filter();
            __syncthreads();
            // the next chunk's codes, in flight during this chunk's MFMAs
            if (ch + KG < nchunks) {
                fetch(ch + KG);
            } else if (c0 + KG >= nchunks && tile + nwg < p.ntm && half < nchunks) {
                prepare(tile + nwg);
                fetch(half);
            }
            if (!active) continue;

            // fragments of tap t (B: channel 32 j + lr; A: the patch pixel of tap t)
            auto frags = [&](int t, v8i (&fa)[NMB], v8i (&fb)[NNB]) {
                const int tr = t / 3, ts = t - 3 * tr;
#pragma unroll
                for (int j = 0; j < NNB; j++) {
                    const uint8_t* b = &wlds[btile + 32 * (nbw + j) * WST + 64 * t];
                    const v4i lo = *(const v4i*)b, hi = *(const v4i*)(b + 16);
                    fb[j] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                }
#pragma unroll
                for (int i = 0; i < NMB; i++) {
                    const int pix = pb[i] + tr * cols + (ts == 0 ? 0 : (ts == 1 ? tcol1 : tcol2));
                    const int a0 = patch_off(pix, 2 * lg);
                    const v4i lo = *(const v4i*)&patch[a0], hi = *(const v4i*)&patch[a0 ^ 16];
                    fa[i] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                }
            };
            // the next tap's fragments are read before this tap's MFMAs are issued, so
            // their LDS latency overlaps the MFMAs (two taps' fragments live at a time)
            v8i fa[NMB], fb[NNB];
            frags(0, fa, fb);
#pragma unroll
            for (int t = 0; t < TAPS; t++) {
                v8i na[NMB], nb[NNB];
                if (t + 1 < TAPS) frags(t + 1, na, nb);
#pragma unroll
                for (int i = 0; i < NMB; i++)
#pragma unroll
                    for (int j = 0; j < NNB; j++)
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                            fb[j], fa[i], acc[i][j], 0, 0, 0, 127, 0, 127);
                __builtin_amdgcn_sched_barrier(0);
                if (t + 1 < TAPS) {
#pragma unroll
                    for (int i = 0; i < NMB; i++) fa[i] = na[i];
#pragma unroll
                    for (int j = 0; j < NNB; j++) fb[j] = nb[j];
                }
            }
        }

        // ---- epilogue: register r of block (i, j) is pixel m0 + 32 (mbw + i) + lr, channel
        //      n0 + 32 (nbw + j) + 8 (r / 4) + 4 lg + r % 4.  Straight from the registers
        //      (store_direct) where the form allows, else the scaled values go through the
        //      wave's LDS slab (rows of 72 floats) and come back as four consecutive channels
        //      per lane, one pixel block at a time.
        if constexpr (KG == 1 && (OUT == 1 || OUT == 2)) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NMB; i++) {
                f32x4 res[4 * NNB];
                const int mrow = m0 + 32 * (mbw + i);
                if (OUT == 1 && p.post.res) load_res<NNB>(p, res, mrow, n0 + 32 * nbw, lane);
                amax = max(amax, store_direct<NNB, OUT>(p, acc[i], res, mrow, n0 + 32 * nbw, lane, s, qa));
            }
            continue;
        }
        __syncthreads();   // every read of the patch is done: the slabs reuse it
        if constexpr (KG == 2 && NNB == 1) {
            // one block per wave: the second half gives its sums to the first
            if (half) {
#pragma unroll
                for (int r = 0; r < 16; r++) ((float*)patch_all[0])[r * kThreads + tid] = acc[0][0][r];
            }
            __syncthreads();
            if (!half) {
#pragma unroll
                for (int r = 0; r < 16; r++) acc[0][0][r] += ((const float*)patch)[r * kThreads + tid];
            }
            __syncthreads();
            if (half) continue;   // the next tile's patch fill starts behind a barrier of all waves
            if constexpr (OUT == 1 || OUT == 2) {
                f32x4 res[4];
                if (OUT == 1 && p.post.res) load_res<1>(p, res, m0 + 32 * mbw, n0 + 32 * nbw, lane);
                amax = max(amax, store_direct<1, OUT>(p, acc[0], res, m0 + 32 * mbw, n0 + 32 * nbw, lane, s, qa));
                continue;
            }
            float* slab = (float*)patch + wave * (32 * SLAB);
            to_slab(slab, SLAB, acc[0][0], 0, lane, s, p.out_shift);
            // a wave reads back only what it wrote
            amax = max(amax, store_block<32, true>(p, slab, SLAB, m0 + 32 * mbw, n0 + 32 * nbw, lane, qa));
            continue;
        } else if constexpr (KG == 2) {
            // each half gives the other one of its two channel blocks, adds what it gets to the
            // block of its own number and stores that
            static_assert(16 * kThreads * 4 <= kPatchMax, "a block of every wave fits the patch");
            float* out = (float*)patch_all[half ^ 1];
            const float* in = (const float*)patch;
#pragma unroll
            for (int r = 0; r < 16; r++) out[r * kThreads + tid] = half ? acc[0][0][r] : acc[0][1][r];
            __syncthreads();
            v16f sum[1];
#pragma unroll
            for (int r = 0; r < 16; r++) sum[0][r] = (half ? acc[0][1][r] : acc[0][0][r]) + in[r * kThreads + tid];
            const int mrow = m0 + 32 * mbw, cc = 32 * half;
            if constexpr (OUT == 1 || OUT == 2) {
                f32x4 res[4];
                if (OUT == 1 && p.post.res) load_res<1>(p, res, mrow, n0 + cc, lane);
                amax = max(amax, store_direct<1, OUT>(p, sum, res, mrow, n0 + cc, lane, s, qa));
                continue;
            }
            __syncthreads();
            float* slab = (float*)patch + wave * (32 * SLAB);
            to_slab(slab, SLAB, sum[0], 0, lane, s, p.out_shift);
            __syncthreads();
            amax = max(amax, store_block<32, true>(p, slab, SLAB, mrow, n0 + cc, lane, qa));
            continue;
        }
        float* slab = (float*)patch + wave * (32 * SLAB);
        constexpr int WCOLS = 32 * NNB;              // channels of a wave's blocks
        const int c0 = 32 * nbw;                      // their first column in the tile
#pragma unroll
        for (int i = 0; i < NMB; i++) {
            const int mrow = m0 + 32 * (mbw + i);
            if (ACC) {   // the exact integer sums, through the slab as well
#pragma unroll
                for (int j = 0; j < NNB; j++) to_slab_int(slab, SLAB, acc[i][j], 32 * j, lane, p.out_shift);
                __syncthreads();
#pragma unroll 1
                for (int e = 4 * lane; e < 32 * WCOLS; e += 256) {
                    const int row = e / WCOLS, col = e - row * WCOLS;
                    const int m = mrow + row;
                    if (m < p.M) {
                        const int4 v = *(const int4*)((const int32_t*)slab + row * SLAB + col);
                        int32_t* d = p.acc + (int64_t)m * p.K + n0 + c0 + col;
                        if (((uintptr_t)d & 15) == 0) {
                            *(int4*)d = v;
                        } else {
                            d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
                        }
                    }
                }
                __syncthreads();
            }
#pragma unroll
            for (int j = 0; j < NNB; j++) to_slab(slab, SLAB, acc[i][j], 32 * j, lane, s, p.out_shift);
            __syncthreads();
            amax = max(amax, store_block<WCOLS, NMB == 1>(p, slab, SLAB, mrow, n0 + c0, lane, qa));
            __syncthreads();
        }
    }
    post_absmax_flush(p.post, amax);
}

// ---------------------------------------------------------------------------
// Resident filter: for more than one chunk of input channels, one workgroup of
// eight waves per CU keeps the filter rows of its output channels (NTR = 64 or
// 32 of them, all 9 C bytes each) decoded in LDS for all of its tiles, so only
// the patch rows travel per chunk.  Tiles of 256 pixels, one 32-pixel block per
// wave; a row of the filter copy is 9 C + 16 bytes (an odd number of 16-byte
// groups: the 16 lanes of a quarter-wave take 16 different bank groups).
constexpr int kResThreads = 512;
constexpr int kResFilterMax = 76 * 1024;   // bytes of the resident filter copy
constexpr int kResFill = 10;               // filter chunks and patch chunks per thread

template <int NNB, int OUT, int FILL>
__global__ __launch_bounds__(kResThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_conv3x3_res(Conv3Params p) {
    constexpr bool ACC = OUT == 3;
    constexpr int NTR = 32 * NNB;              // output channels per workgroup
    constexpr int TM = 256;                    // pixels per tile: block `wave` of 8
    constexpr int SL = NTR + 8;                // slab row stride (floats): two lane halves
                                               // 4 rows apart are 32 banks apart
    static_assert(4 * 32 * SL * 4 <= kPatchMax, "epilogue slabs fit");
    __shared__ __align__(16) uint8_t wres[kResFilterMax];
    __shared__ __align__(16) uint8_t patch[kPatchMax];
    __shared__ __align__(16) uint8_t spare[kPatchMax];   // the slabs of waves 4..7
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, lg = lane >> 5;

    const int nt = (int)blockIdx.x % p.ntn;
    const int n0 = nt * NTR;
    const int wg = (int)blockIdx.x / p.ntn, nwg = (int)gridDim.x / p.ntn;
    const int nchunks = p.C / CK;
    const int wst = TAPS * p.C + 16;                      // LDS bytes per filter row
    const int row16 = TAPS * p.C / 16;                    // 16-byte chunks of a filter row

    // ---- the filter rows n0 .. n0 + NTR - 1, once, every load in flight
    {
        uint4 wv[kResFill];
#pragma unroll
        for (int u = 0; u < kResFill; u++) {
            const int it = tid + u * kResThreads;
            const int k = it / row16, rem = it - k * row16;
            wv[u] = k < NTR ? *(const uint4*)(p.w + (int64_t)(n0 + k) * (TAPS * p.C) + 16 * rem)
                            : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int u = 0; u < kResFill; u++) {
            const int it = tid + u * kResThreads;
            const int k = it / row16, rem = it - k * row16;
            if (k < NTR) *(uint4*)&wres[k * wst + 16 * rem] = dec16(wv[u], p.dw);
        }
    }

    float s = 0.0f;   // int32 sums alone: the scales may be NULL
    if (!ACC || p.y || p.post.on) s = ldexpf(p.alphaX[0] * p.alphaW[0], -(p.kX + p.kW));
    const float qa = post_alpha(p.post);
    uint32_t amax = 0;
    const int cols = p.Q + 2, PP2 = p.P + 2, PQ = p.P * p.Q;
    const int cpr = 4 * cols;
    const int fci = tid % cpr, fri = tid / cpr, rstep = kResThreads / cpr;
    const int fcol = fci >> 2, fc = fci & 3, iw = fcol - 1;
    const bool col_in = (unsigned)iw < (unsigned)p.Q;
    // B fragments: output channel 32 j + lr, bytes 32 lg .. + 31 of (tap t, chunk ch)
    const int boff = lr * wst + 32 * lg;

    auto rows_of = [&](int tile, int& R0, int& nrows) {
        const int m0 = tile * TM;
        const int i0 = m0 / PQ, p0 = (m0 - i0 * PQ) / p.Q;
        R0 = i0 * PP2 + p0;
        const int m1 = min(m0 + TM, p.M) - 1;
        const int i1 = m1 / PQ, p1 = (m1 - i1 * PQ) / p.Q;
        nrows = i1 * PP2 + p1 + 3 - R0;
    };
    uint4 raw[FILL];   // as in k_conv3x3
    uint32_t poff[FILL], vmask = 0;
    int frows = 0;
    auto prepare = [&](int tile) {
        int R0;
        rows_of(tile, R0, frows);
        const int pr = R0 + fri;
        int n = pr / PP2, hp = pr - n * PP2;
        vmask = 0;
#pragma unroll
        for (int u = 0; u < FILL; u++) {
            const int ih = hp - 1;
            const bool ok = fri < rstep && fri + u * rstep < frows && col_in && n < p.N &&
                            (unsigned)ih < (unsigned)p.P;
            poff[u] = (ok ? ((uint32_t)(n * p.P + ih) * p.Q + iw) * (uint32_t)p.C : 0u) + 16 * fc;
            vmask |= ok ? (1u << u) : 0u;
            hp += rstep;
            while (hp >= PP2) { hp -= PP2; n++; }
        }
    };
    auto fetch = [&](int ch) {
        const uint8_t* xc = p.x + CK * ch;
#pragma unroll
        for (int u = 0; u < FILL; u++) {
            raw[u] = *(const uint4*)(xc + poff[u]);
        }
    };
    if (wg < p.ntm) {
        prepare(wg);
        fetch(0);
    }

    for (int tile = wg; tile < p.ntm; tile += nwg) {
        const int m0 = tile * TM;
        int R0, nrows;
        rows_of(tile, R0, nrows);
        int pb;
        {
            const int m = min(m0 + 32 * wave + lr, p.M - 1);   // rows past M: any pixel
            const int n = m / PQ, rem = m - n * PQ;
            const int pp = rem / p.Q, q = rem - pp * p.Q;
            pb = (n * PP2 + pp - R0) * cols + q;
        }
        v16f acc[NNB];
#pragma unroll
        for (int j = 0; j < NNB; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[j][r] = 0.0f;

        for (int ch = 0; ch < nchunks; ch++) {
            __syncthreads();   // the previous chunk's (or tile's) reads of the patch are done
            if (fri < rstep) {
#pragma unroll
                for (int u = 0; u < FILL; u++) {
                    const int i = fri + u * rstep;
                    if (i < frows) {
                        const uint4 v = ((vmask >> u) & 1u) ? dec16(raw[u], p.dx)
                                                            : make_uint4(0u, 0u, 0u, 0u);   // E4M3 +0
                        *(uint4*)&patch[patch_off(i * cols + fcol, fc)] = v;
                    }
                }
            }
            __syncthreads();
            if (ch + 1 < nchunks) {
                fetch(ch + 1);
            } else if (tile + nwg < p.ntm) {
                prepare(tile + nwg);
                fetch(0);
            }

            const uint8_t* wb = &wres[boff + CK * ch];
            auto frags = [&](int t, v8i& fa, v8i (&fb)[NNB]) {
                const int tr = t / 3, ts = t - 3 * tr;
#pragma unroll
                for (int j = 0; j < NNB; j++) {
                    const uint8_t* b = wb + 32 * j * wst + t * p.C;
                    const v4i lo = *(const v4i*)b, hi = *(const v4i*)(b + 16);
                    fb[j] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                }
                const int pix = pb + tr * cols + ts;
                const int a0 = patch_off(pix, 2 * lg);
                const v4i lo = *(const v4i*)&patch[a0], hi = *(const v4i*)&patch[a0 ^ 16];
                fa = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            };
            v8i fa, fb[NNB];   // the next tap's fragments read before this tap's MFMAs
            frags(0, fa, fb);
#pragma unroll
            for (int t = 0; t < TAPS; t++) {
                v8i na, nb[NNB];
                if (t + 1 < TAPS) frags(t + 1, na, nb);
#pragma unroll
                for (int j = 0; j < NNB; j++)
                    acc[j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        fb[j], fa, acc[j], 0, 0, 0, 127, 0, 127);
                __builtin_amdgcn_sched_barrier(0);
                if (t + 1 < TAPS) {
                    fa = na;
#pragma unroll
                    for (int j = 0; j < NNB; j++) fb[j] = nb[j];
                }
            }
        }

        // ---- epilogue of block `wave` (pixels m0 + 32 wave ..), as in k_conv3x3
        if constexpr (OUT == 1 || OUT == 2) {
            f32x4 res[4 * NNB];
            if (OUT == 1 && p.post.res) load_res<NNB>(p, res, m0 + 32 * wave, n0, lane);
            amax = max(amax, store_direct<NNB, OUT>(p, acc, res, m0 + 32 * wave, n0, lane, s, qa));
            continue;
        }
        __syncthreads();   // every read of the patch is done: the slabs reuse it
        float* slab = (float*)(wave < 4 ? patch : spare) + (wave & 3) * (32 * SL);
        const int mrow = m0 + 32 * wave;
        if (ACC) {
#pragma unroll
            for (int j = 0; j < NNB; j++) to_slab_int(slab, SL, acc[j], 32 * j, lane, p.out_shift);
            __syncthreads();
#pragma unroll 1
            for (int e = 4 * lane; e < 32 * NTR; e += 256) {
                const int row = e / NTR, col = e - row * NTR;
                const int m = mrow + row;
                if (m < p.M) {
                    const int4 v = *(const int4*)((const int32_t*)slab + row * SL + col);
                    int32_t* d = p.acc + (int64_t)m * p.K + n0 + col;
                    if (((uintptr_t)d & 15) == 0) {
                        *(int4*)d = v;
                    } else {
                        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
                    }
                }
            }
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < NNB; j++) to_slab(slab, SL, acc[j], 32 * j, lane, s, p.out_shift);
        __syncthreads();
        amax = max(amax, store_block<NTR, true>(p, slab, SL, mrow, n0, lane, qa));
    }
    post_absmax_flush(p.post, amax);
}

// Output channels per workgroup of the resident-filter kernel (64, else 32), 0
// when neither copy fits.
int res_ntr(int C, int K) {
    for (int ntr = 64; ntr >= 32; ntr >>= 1)
        if (K % ntr == 0 && (int64_t)ntr * (TAPS * C + 16) <= kResFilterMax &&
            (int64_t)ntr * TAPS * C <= (int64_t)kResFill * 16 * kResThreads)
            return ntr;
    return 0;
}

bool res_tile_fits(int P, int Q) {
    if (4 * (Q + 2) > kResThreads) return false;
    const int rstep = kResThreads / (4 * (Q + 2));
    const int dg = (Q - 1 + 256 - 1) / Q, cross = (P - 1 + dg) / P;
    const int rows = dg + 2 * cross + 3;
    return (rows + rstep - 1) / rstep <= kResFill && (int64_t)rows * (Q + 2) * 64 <= kPatchMax;
}

// Rows of the patch of a tile of TM pixels: the padded rows from the first
// pixel's to two past the last pixel's, at most dg + 2 (images crossed) + 3
// rows with dg the output rows a tile spans beyond its first.
// With stride st the tile's output rows span st dg + 3 padded input rows, and each
// image boundary crossed adds the H + 2 - st P padded rows past the last output row's.
int patch_rows_max(int P, int Q, int TM, int H, int st) {
    const int dg = (Q - 1 + TM - 1) / Q;
    const int cross = (P - 1 + dg) / P;
    return st * dg + cross * (H + 2 - st * P) + 3;
}

bool tile_fits(int P, int Q, int TM, int H, int W, int st) {
    if (W + 2 > kMaxCols) return false;
    const int rstep = kThreads / (4 * (W + 2));
    const int rows = patch_rows_max(P, Q, TM, H, st);
    return (rows + rstep - 1) / rstep <= kMaxFill && (int64_t)rows * (W + 2) * 64 <= kPatchMax;
}

// 32-pixel blocks per tile: the largest of 8, 4, 2 (4, 2 with several chunks of
// input channels) whose tiles fit the patch and give at least one workgroup per
// CU (half a workgroup per CU with several chunks: every tile streams the filter
// slices again, so larger tiles halve that traffic per pixel; ResNet18 l4 at batch
// 64, 200 tiles of 128 pixels against 392 of 64: 20.7 against 26.4 us), else the
// smallest: one 56 x 56 image with 64 channels takes 10.4 us in 13 tiles of 256
// pixels and 7.2 in 49 of 64, 256 channels at 14 x 14 16.2 and 13.7.
int choose_tmb(int64_t M, int ntn, int P, int Q, int H, int W, int st, bool multi) {
    const int cus = num_cus();
    int fit = 0;
    for (int tmb = multi ? 4 : 8; tmb >= 2; tmb >>= 1) {
        if (!tile_fits(P, Q, 32 * tmb, H, W, st)) continue;
        fit = tmb;
        if ((M + 32 * tmb - 1) / (32 * tmb) * ntn >= (multi ? cus / 2 : cus)) return tmb;
    }
    return fit;
}

}  // namespace

// Images per launch: the kernels keep places in the input in 32 bits, so that larger inputs
// (4 GiB and more) run in equal parts of whole images (4.3 GB of 256 channels at 56 x 56 -> 64:
// 4.57 ms, on the implicit-GEMM kernels 6.80).  0: a single image is too large.
static int images_per_launch(const ConvGeom& g) {
    const int64_t image = (int64_t)g.H * g.W * g.C, most = ((int64_t)1 << 32) - 1;
    if (image > most) return 0;
    const int64_t fit = image > 0 ? most / image : g.Nb;
    if (fit >= g.Nb) return g.Nb;
    const int64_t parts = (g.Nb + fit - 1) / fit;
    return (int)((g.Nb + parts - 1) / parts);
}

bool conv3x3_fits(const ConvGeom& g, int K, int groups, int op, const uint8_t* x,
                  const uint8_t* w) {
    if (!(groups == 1 && op == 1 && K % NT == 0 && K >= NT && g.C % CK == 0 && g.C >= CK &&
          g.Cg == g.C && g.pitch == g.C && g.R == 3 && g.S == 3 && g.ph == 1 && g.pw == 1 &&
          g.P >= 1 && g.Q >= 1))
        return false;
    const bool s1 = g.sh == 1 && g.sw == 1 && g.P == g.H && g.Q == g.W;
    const bool s2 = g.sh == 2 && g.sw == 2 && g.P == (g.H - 1) / 2 + 1 && g.Q == (g.W - 1) / 2 + 1;
    if (!s1 && !s2) return false;
    // Stride 2 takes tiles of 64 output pixels (the patch holds four times the input
    // of stride 1 per pixel), whose fill, repeated by every tile of 64 output channels,
    // outweighs the MFMAs unless the input channels run to several chunks: measured
    // at batch 64 against the implicit-GEMM path, 256 -> 512 at 14 x 14 24.1 against
    // 28.4 us, but 64 -> 128 at 56 x 56 25.3 against 21.0 and 128 -> 256 at 28 x 28
    // 28.5 against 19.6.
    if (s2 && g.C < 4 * CK) return false;
    if ((uintptr_t)x % 16 || (uintptr_t)w % 16) return false;
    const int64_t M = (int64_t)g.Nb * g.P * g.Q;
    if ((M + 256) * K >= ((int64_t)1 << 31) || (int64_t)K * TAPS * g.C >= ((int64_t)1 << 31)) return false;
    const int per = images_per_launch(g);
    if (per < g.Nb) {
        if (per == 0) return false;
        ConvGeom part = g;
        part.Nb = per;
        if (!conv3x3_fits(part, K, groups, op, x, w)) return false;
        part.Nb = g.Nb % per;
        return part.Nb == 0 || conv3x3_fits(part, K, groups, op, x, w);
    }
    // With several chunks every workgroup decodes its 64 filter rows per chunk and tile:
    // measured faster than the implicit-GEMM kernels only for few output pixels (ResNet18
    // 3x3 at batch 64: 256 channels at 14 x 14 and 512 at 7 x 7 faster, 128 at 28 x 28
    // with 50176 pixels slower).
    if (g.C > CK && M > kMultiMaxPixels)   // several chunks and many pixels: resident filter
        return s1 && res_ntr(g.C, K) != 0 && res_tile_fits(g.P, g.Q);
    return choose_tmb(M, K / NT, g.P, g.Q, g.H, g.W, g.sh, g.C > CK) != 0;
}

hipError_t launch_conv3x3(const ConvGeom& g, int K, const uint8_t* x, const Fmt& fx,
                          const float* alphaX, const uint8_t* w, const Fmt& fw,
                          const float* alphaW, int32_t* acc, float* y, hipStream_t s,
                          const Post* post) {
    const int images = images_per_launch(g);
    if (images < g.Nb) {
        if (images == 0) return hipErrorInvalidValue;
        for (int n0 = 0; n0 < g.Nb; n0 += images) {
            ConvGeom part = g;
            part.Nb = g.Nb - n0 < images ? g.Nb - n0 : images;
            const int64_t o = (int64_t)n0 * g.P * g.Q * K;
            Post P;
            if (post) {
                P = *post;
                if (P.res) P.res += o;
                if (P.codes) P.codes += o;
            }
            const hipError_t e = launch_conv3x3(part, K, x + (int64_t)n0 * g.H * g.W * g.C, fx, alphaX, w, fw,
                                                alphaW, acc ? acc + o : nullptr, y ? y + o : nullptr, s,
                                                post ? &P : nullptr);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    Conv3Params p{};
    p.x = x;
    p.w = w;
    p.alphaX = alphaX;
    p.alphaW = alphaW;
    p.acc = acc;
    p.y = y;
    p.dx = mma_decode(fx, 1);
    p.dw = mma_decode(fw, 1);
    if (post) p.post = *post;
    p.N = g.Nb;
    p.P = g.P;
    p.Q = g.Q;
    p.H = g.H;
    p.W = g.W;
    p.st = g.sh;
    p.half = (g.W + 3) / 2;
    p.M = g.Nb * g.P * g.Q;
    p.C = g.C;
    p.K = K;
    if (p.M == 0) return hipSuccess;
    p.out_shift = fx.k + fw.k + 12;
    p.kX = fx.k;
    p.kW = fw.k;
    if (!acc && !p.post.a && !p.post.b) {   // K is a multiple of 64: every row starts aligned
        if (y && !p.post.codes && (uintptr_t)y % 16 == 0 && (uintptr_t)p.post.res % 16 == 0) p.direct = 1;
        if (!y && p.post.codes && !p.post.res && (uintptr_t)p.post.codes % 16 == 0) p.direct = 2;
    }
    // The resident-filter kernel, one workgroup per CU: several chunks and many pixels; one
    // chunk too where codes leave (its outputs go straight from the registers, the two-
    // workgroup kernel's through slabs: 64 -> 64 at 56 x 56, batch 64, 35.5 against 27.4 us;
    // fp32 outputs 24.6 against 29.5, four times the bytes behind one workgroup).
    const bool one_res = g.C == CK && p.direct == 2 && p.st == 1 && res_ntr(g.C, K) != 0 &&
                         res_tile_fits(g.P, g.Q);
    if ((g.C > CK || one_res) && p.M > kMultiMaxPixels) {
        if (p.st != 1) return hipErrorInvalidValue;
        const int ntr = res_ntr(g.C, K);
        if (ntr == 0 || !res_tile_fits(g.P, g.Q)) return hipErrorInvalidValue;
        p.ntn = K / ntr;
        p.ntm = (p.M + 255) / 256;
        int per = num_cus() / p.ntn;
        if (per < 1) per = 1;
        if (per > p.ntm) per = p.ntm;
        const unsigned blocks = (unsigned)(per * p.ntn);
        const int rs = kResThreads / (4 * (g.Q + 2));
        const bool few = (patch_rows_max(g.P, g.Q, 256, g.H, 1) + rs - 1) / rs <= kFewFill;
#define ESB_CONV3_LAUNCH(NNB, FILL)                                                       \
    do {                                                                                  \
        if (acc) k_conv3x3_res<NNB, 3, FILL><<<blocks, kResThreads, 0, s>>>(p);           \
        else if (p.direct == 1) k_conv3x3_res<NNB, 1, FILL><<<blocks, kResThreads, 0, s>>>(p); \
        else if (p.direct == 2) k_conv3x3_res<NNB, 2, FILL><<<blocks, kResThreads, 0, s>>>(p); \
        else k_conv3x3_res<NNB, 0, FILL><<<blocks, kResThreads, 0, s>>>(p);               \
    } while (0)
        if (ntr == 64 && few) ESB_CONV3_LAUNCH(2, kFewFill);
        else if (ntr == 64) ESB_CONV3_LAUNCH(2, kResFill);
        else if (few) ESB_CONV3_LAUNCH(1, kFewFill);
        else ESB_CONV3_LAUNCH(1, kResFill);
#undef ESB_CONV3_LAUNCH
        return hipGetLastError();
    }
    p.ntn = K / NT;
    const bool multi = g.C > CK;
    const int tmb = choose_tmb(p.M, p.ntn, g.P, g.Q, g.H, g.W, p.st, multi);
    if (tmb == 0) return hipErrorInvalidValue;
    p.ntm = (p.M + 32 * tmb - 1) / (32 * tmb);
    // patch chunks per thread: 5 where they suffice (most images of up to 30 columns), else more
    const int rstep = kThreads / (4 * (g.W + 2));
    const int fill = (patch_rows_max(g.P, g.Q, 32 * tmb, g.H, p.st) + rstep - 1) / rstep;
    const bool few = fill <= kFewFill;
    // the reduction in two halves (see k_conv3x3): one tile per CU at most, six chunks or more
    if (!acc && g.C >= 6 * CK && (int64_t)p.ntm * p.ntn <= num_cus()) {
        const unsigned blocks = (unsigned)(p.ntm * p.ntn);
#define ESB_CONV3_LAUNCH(TMB, FILL)                                                                   \
    do {                                                                                              \
        if (p.direct == 1) k_conv3x3<TMB, true, 1, FILL, 2><<<blocks, 2 * kThreads, 0, s>>>(p);       \
        else if (p.direct == 2) k_conv3x3<TMB, true, 2, FILL, 2><<<blocks, 2 * kThreads, 0, s>>>(p);  \
        else k_conv3x3<TMB, true, 0, FILL, 2><<<blocks, 2 * kThreads, 0, s>>>(p);                     \
    } while (0)
        if (tmb == 4 && few) ESB_CONV3_LAUNCH(4, kFewFill);
        else if (tmb == 4) ESB_CONV3_LAUNCH(4, kMaxFill);
        else if (few) ESB_CONV3_LAUNCH(2, kFewFill);
        else ESB_CONV3_LAUNCH(2, kMaxFill);
#undef ESB_CONV3_LAUNCH
        return hipGetLastError();
    }
    // Wide images, whose tiles of 128 pixels take more than five patch chunks per thread, have no
    // registers for the residual beside those of the next chunk: 128 -> 384 at 60 x 60, batch 4,
    // 33.0 us straight from the accumulators with room for ten chunks (48 registers spilled), 27.6
    // through the slabs with room for nine (12 spilled).
    if (multi && tmb == 4 && !few && p.post.res) p.direct = 0;
    // persistent workgroups, a whole number per channel tile, two per CU
    int per = (num_cus() * 2) / p.ntn;
    if (per < 1) per = 1;
    if (per > p.ntm) per = p.ntm;
    const unsigned blocks = (unsigned)(per * p.ntn);
    // (one chunk with tiles of 128 pixels or more keeps the slabs: its direct instances spill)
#define ESB_CONV3_LAUNCH2(TMB, MULTI, FILL)                                                    \
    do {                                                                                       \
        constexpr bool D = MULTI || TMB == 2;                                                  \
        if (acc) k_conv3x3<TMB, MULTI, 3, FILL><<<blocks, kThreads, 0, s>>>(p);                \
        else if (D && p.direct == 1) k_conv3x3<TMB, MULTI, D ? 1 : 0, FILL><<<blocks, kThreads, 0, s>>>(p); \
        else if (D && p.direct == 2) k_conv3x3<TMB, MULTI, D ? 2 : 0, FILL><<<blocks, kThreads, 0, s>>>(p); \
        else k_conv3x3<TMB, MULTI, 0, FILL><<<blocks, kThreads, 0, s>>>(p);                    \
    } while (0)
#define ESB_CONV3_LAUNCH(TMB, MULTI)                                                 \
    do {                                                                             \
        if (few) ESB_CONV3_LAUNCH2(TMB, MULTI, kFewFill);                            \
        else ESB_CONV3_LAUNCH2(TMB, MULTI, kMaxFill);                                \
    } while (0)
    if (!multi && tmb == 8) ESB_CONV3_LAUNCH2(8, false, kMaxFill);   // its tiles have six rows of chunks and more
    else if (!multi && tmb == 4) ESB_CONV3_LAUNCH(4, false);
    else if (!multi) ESB_CONV3_LAUNCH(2, false);
    else if (tmb == 4 && acc && !few && fill <= kSumsFill)
        k_conv3x3<4, true, 3, kSumsFill><<<blocks, kThreads, 0, s>>>(p);
    else if (tmb == 4 && !few && fill <= kMidFill) ESB_CONV3_LAUNCH2(4, true, kMidFill);
    else if (tmb == 4) ESB_CONV3_LAUNCH(4, true);
    else ESB_CONV3_LAUNCH(2, true);
#undef ESB_CONV3_LAUNCH
#undef ESB_CONV3_LAUNCH2
    return hipGetLastError();
}

}  // namespace esb
