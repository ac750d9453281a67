// Depthwise convolution over ESB codes (groups == C == K, one filter per
// channel), gfx950.  R*S multiply-adds per output: far below the MFMA ridge, so
// these are VALU kernels (codes in, int32 / fp32 out); at MobileNet sizes the
// byte extraction, table lookups and multiply-adds bound them, not HBM.
// k_dw3: 3x3 / stride 1, four channels and four columns per thread walking down
// a strip of rows, byte dot products (formats of at most five bits);
// k_dwconv16: sixteen channels of one output pixel per thread (C % 16 == 0);
// k_dwconv: four channels (C % 4 == 0) or one.  In the last two decoded filter
// taps live in LDS as int16, activation codes are decoded through a 256-entry
// LDS table of exact integers.
#include "esb_internal.h"

namespace esb {

struct DwParams {
    ConvGeom g;
    const uint8_t* x;
    const uint8_t* w;
    const float* alphaX;
    const float* alphaW;
    int32_t* acc;
    float* y;
    int kx, kw;
    Post post;         // fused post-processing of the outputs (post.on == 0: none)
    int16_t tx[256];   // exact integer of every activation code
    int16_t tw[256];   // exact integer of every filter code
};

constexpr int kDwThreads = 256;
constexpr int kDwMaxTaps = 16384;   // C * R * S held in LDS

template <bool VEC>
__global__ __launch_bounds__(kDwThreads) void k_dwconv(DwParams p) {
    __shared__ int16_t wt[kDwMaxTaps];
    __shared__ int tx[256];
    const ConvGeom& g = p.g;
    const int C = g.C, RS = g.R * g.S;
    for (int i = threadIdx.x; i < C * RS; i += blockDim.x) wt[i] = p.tw[p.w[i]];
    tx[threadIdx.x] = p.tx[threadIdx.x];
    __syncthreads();
    float s = 0.0f;
    if (p.y || p.post.on) s = ldexpf(p.alphaX[0] * p.alphaW[0], -(p.kx + p.kw));
    const float qa = p.post.on ? post_alpha(p.post) : 0.0f;
    const int CV = VEC ? C / 4 : C;                 // channel groups per pixel
    const int64_t total = (int64_t)g.Nb * g.P * g.Q * CV;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    uint32_t amax = 0;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += stride) {
        const int cv = (int)(t % CV);
        const int64_t pix = t / CV;
        const int q = (int)(pix % g.Q);
        const int p_ = (int)((pix / g.Q) % g.P);
        const int n = (int)(pix / ((int64_t)g.Q * g.P));
        const int c0 = VEC ? 4 * cv : cv;
        int a0 = 0, a1 = 0, a2 = 0, a3 = 0;
        for (int r = 0; r < g.R; r++) {
            const int ih = p_ * g.sh - g.ph + r;
            if (ih < 0 || ih >= g.H) continue;
            for (int s2 = 0; s2 < g.S; s2++) {
                const int iw = q * g.sw - g.pw + s2;
                if (iw < 0 || iw >= g.W) continue;
                const int64_t base = (((int64_t)n * g.H + ih) * g.W + iw) * C + c0;
                const int tap = r * g.S + s2;
                if (VEC) {
                    const uint32_t w4 = *(const uint32_t*)(p.x + base);
                    a0 += tx[w4 & 0xff] * wt[(c0 + 0) * RS + tap];
                    a1 += tx[(w4 >> 8) & 0xff] * wt[(c0 + 1) * RS + tap];
                    a2 += tx[(w4 >> 16) & 0xff] * wt[(c0 + 2) * RS + tap];
                    a3 += tx[w4 >> 24] * wt[(c0 + 3) * RS + tap];
                } else {
                    a0 += tx[p.x[base]] * wt[c0 * RS + tap];
                }
            }
        }
        const int64_t o = pix * C + c0;
        if (VEC) {
            if (p.acc) *(int4*)(p.acc + o) = make_int4(a0, a1, a2, a3);
            if (p.post.on) {
                amax = max(amax, post_store(p.post, p.y, o, c0, s * (float)a0, qa));
                amax = max(amax, post_store(p.post, p.y, o + 1, c0 + 1, s * (float)a1, qa));
                amax = max(amax, post_store(p.post, p.y, o + 2, c0 + 2, s * (float)a2, qa));
                amax = max(amax, post_store(p.post, p.y, o + 3, c0 + 3, s * (float)a3, qa));
            } else if (p.y) {
                *(float4*)(p.y + o) = make_float4(s * (float)a0, s * (float)a1, s * (float)a2,
                                                  s * (float)a3);
            }
        } else {
            if (p.acc) p.acc[o] = a0;
            amax = max(amax, out_store(p.post, p.y, o, c0, s * (float)a0, qa));
        }
    }
    post_absmax_flush(p.post, amax);
}

// Sixteen channels per thread (C % 16 == 0, at most 16 filter taps): one 16-byte
// load of codes per tap, the taps' weights read as 32-byte rows of an LDS table
// laid out [tap][channel], four 16-byte stores per output.  The grid is sized so
// that the grid-stride step is a multiple of C / 16: every thread keeps one
// channel group and walks output pixels.
constexpr int kDw16MaxTaps = 16;
__global__ __launch_bounds__(kDwThreads) void k_dwconv16(DwParams p, int pix_step) {
    __shared__ __align__(16) int16_t wt[kDwMaxTaps];   // [tap][channel]
    __shared__ int tx[256];
    const ConvGeom& g = p.g;
    const int C = g.C, RS = g.R * g.S, CV = C / 16;
    for (int i = threadIdx.x; i < C * RS; i += blockDim.x) {
        const int c = i / RS, tap = i - c * RS;                  // KRSC: channel-major source
        wt[tap * C + c] = p.tw[p.w[i]];
    }
    tx[threadIdx.x] = p.tx[threadIdx.x];
    __syncthreads();
    float s = 0.0f;
    if (p.y || p.post.on) s = ldexpf(p.alphaX[0] * p.alphaW[0], -(p.kx + p.kw));
    const float qa = p.post.on ? post_alpha(p.post) : 0.0f;
    const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int cv = (int)(gt % CV), c0 = 16 * cv;
    const int64_t npix = (int64_t)g.Nb * g.P * g.Q;
    uint32_t amax = 0;
    for (int64_t pix = gt / CV; pix < npix; pix += pix_step) {
        const int q = (int)(pix % g.Q);
        const int p_ = (int)((pix / g.Q) % g.P);
        const int n = (int)(pix / ((int64_t)g.Q * g.P));
        int a[16];
#pragma unroll
        for (int e = 0; e < 16; e++) a[e] = 0;
        for (int r = 0; r < g.R; r++) {
            const int ih = p_ * g.sh - g.ph + r;
            if (ih < 0 || ih >= g.H) continue;
            for (int s2 = 0; s2 < g.S; s2++) {
                const int iw = q * g.sw - g.pw + s2;
                if (iw < 0 || iw >= g.W) continue;
                const uint4 cx = *(const uint4*)(p.x + (((int64_t)n * g.H + ih) * g.W + iw) * C + c0);
                const int tap = r * g.S + s2;
                const int4* wr = (const int4*)(wt + tap * C + c0);
                const int4 w0 = wr[0], w1 = wr[1];
                const uint32_t cw[4] = {cx.x, cx.y, cx.z, cx.w};
                const uint32_t ww[8] = {(uint32_t)w0.x, (uint32_t)w0.y, (uint32_t)w0.z, (uint32_t)w0.w,
                                        (uint32_t)w1.x, (uint32_t)w1.y, (uint32_t)w1.z, (uint32_t)w1.w};
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const int xv = tx[(cw[e >> 2] >> (8 * (e & 3))) & 0xffu];
                    const int wv = (int)(int16_t)(ww[e >> 1] >> (16 * (e & 1)));
                    a[e] += xv * wv;
                }
            }
        }
        const int64_t o = pix * C + c0;
        if (p.acc) {
#pragma unroll
            for (int k = 0; k < 4; k++)
                *(int4*)(p.acc + o + 4 * k) = make_int4(a[4 * k], a[4 * k + 1], a[4 * k + 2], a[4 * k + 3]);
        }
        if (p.post.on) {
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const f32x4 v{s * (float)a[4 * k], s * (float)a[4 * k + 1], s * (float)a[4 * k + 2],
                              s * (float)a[4 * k + 3]};
                amax = max(amax, post_store4(p.post, p.y, o + 4 * k, c0 + 4 * k, v, 4, qa));
            }
        } else if (p.y) {
#pragma unroll
            for (int k = 0; k < 4; k++)
                *(float4*)(p.y + o + 4 * k) = make_float4(s * (float)a[4 * k], s * (float)a[4 * k + 1],
                                                          s * (float)a[4 * k + 2], s * (float)a[4 * k + 3]);
        }
    }
    post_absmax_flush(p.post, amax);
}

// 3x3, stride 1, C % 4 == 0, activation formats of at most five bits (decoded four at a
// time by byte permutes), filter integers in int8.  A thread owns four channels (one dword
// of codes per pixel) of four output columns and walks down `rows` output rows: each
// input row is six dwords, decoded once for the three output rows and up to three columns
// that read it, transposed with byte permutes so that one dword holds four neighbouring
// columns of one channel.  That dword serves two output columns by v_dot4_i32_i8 with the
// filter row at bytes 0-2 or 1-3, so an output costs 3 dot products, 1 permute and its share
// (6/4) of a decode instead of 9 table lookups, extractions and multiply-adds.  The three
// output rows in flight rotate through the dot products' addend, without moves.
// MobileNetV2's 3x3 on 144 channels, batch 32, 56x56, codes out: 54.2 us on k_dwconv16
// (48 with the faster codes), 22.3 here; VALU bound.  Shorter strips fill the chip but reread
// two rows each: 16 / 8 / 4 / 2 rows 32 / 25 / 24 / 27 us there.
struct Dw3Params {
    ConvGeom g;
    const uint8_t* x;
    const uint8_t* w;
    const float* alphaX;
    const float* alphaW;
    int32_t* acc;
    float* y;
    DecodeInfo dx, dw;
    uint32_t zero4;       // four +0 codes
    int rows, strips, cols;   // output rows per strip, strips per image, column groups per row
    int total;            // threads with work
    Post post;
};

// Unaligned dword (the filter rows start at any byte).
struct __attribute__((packed)) U32Any { uint32_t v; };

// OUT 0: every epilogue; OUT 1 (fp32 outputs) and OUT 2 (codes): the forms without affine,
// residual or int32 sums, whose stores come in a fixed number per row.  Vector memory
// operations retire in order on one counter, so with a known number of stores after the
// next row's loads the wait for those loads leaves the stores in flight; a store behind a
// branch makes every row wait for its own stores.  For the same reason ragged edges
// overlap instead of branching there: the last column group starts at Q - 4, and threads past
// the end repeat the last one's work (the same values are written twice).
template <int OUT, int MODE>
__global__ __launch_bounds__(kDwThreads) void k_dw3(Dw3Params p) {
    const ConvGeom& g = p.g;
    const int C = g.C, CV = C / 4;
    const int gt = (int)blockIdx.x * kDwThreads + (int)threadIdx.x;
    const bool live = OUT != 0 || gt < p.total;
    unsigned t = (unsigned)min(gt, p.total - 1);
    const int c0 = 4 * (int)(t % (unsigned)CV);
    t /= (unsigned)CV;
    int q0 = 4 * (int)(t % (unsigned)p.cols);
    if (OUT) q0 = min(q0, g.Q - 4);
    t /= (unsigned)p.cols;
    const int r0 = p.rows * (int)(t % (unsigned)p.strips);
    const int n = (int)(t / (unsigned)p.strips);
    const int r1 = live ? min(r0 + p.rows, g.P) : r0;
    // the six input columns of a row: every load issued, at a clamped place, and +0 codes
    // put in where it lies outside the image (by masks: no branches around the loads)
    const uint8_t* xi = p.x + (int64_t)n * g.H * g.W * C + c0;
    int coff[6];
    uint32_t cmask[6];
#pragma unroll
    for (int i = 0; i < 6; i++) {
        const int iw = q0 - g.pw + i;
        coff[i] = min(max(iw, 0), g.W - 1) * C;
        cmask[i] = (unsigned)iw < (unsigned)g.W ? 0xffffffffu : 0u;
    }
    uint32_t rmask = 0u;   // of the row in nx
    auto load_row = [&](int ih, uint32_t (&v)[6]) {
        const bool in_h = (unsigned)ih < (unsigned)g.H;
        const uint8_t* xr = xi + (int64_t)(in_h ? ih : 0) * g.W * C;
        rmask = in_h ? 0xffffffffu : 0u;
#pragma unroll
        for (int i = 0; i < 6; i++) v[i] = *(const uint32_t*)(xr + coff[i]);
    };
    uint32_t nx[6];
    load_row(r0 - g.ph, nx);
    // filter rows of the four channels: {w0, w1, w2, 0} and the same one byte up
    uint32_t wlo[3][4], whi[3][4];
    {
        uint32_t d[10];
#pragma unroll
        for (int i = 0; i < 9; i++) d[i] = ((const U32Any*)(p.w + (int64_t)c0 * 9 + 4 * i))->v;
        __builtin_amdgcn_sched_barrier(0);   // every load in flight before the first decode
        if (p.dw.mode == MODE) {
#pragma unroll
            for (int i = 0; i < 9; i++) d[i] = decode4_lut<MODE>(d[i], p.dw);
        } else {
#pragma unroll
            for (int i = 0; i < 9; i++) d[i] = decode4(d[i], p.dw);
        }
        d[9] = 0u;
#pragma unroll
        for (int c = 0; c < 4; c++)
#pragma unroll
            for (int r = 0; r < 3; r++) {
                const int o = 9 * c + 3 * r;
                const uint32_t v =
                    __builtin_amdgcn_alignbyte(d[o / 4 + 1], d[o / 4], (uint32_t)(o % 4)) & 0xffffffu;
                wlo[r][c] = v;
                whi[r][c] = v << 8;
            }
    }
    float s = 0.0f;
    if (p.y || p.post.on) s = ldexpf(p.alphaX[0] * p.alphaW[0], -(p.dx.k + p.dw.k));
    const float qa = p.post.on ? post_alpha(p.post) : 0.0f;
    const bool q_ok = alpha_valid(qa), q_fast = fast_scale(qa);
    const float q_r = 1.0f / qa;
    int a1[4][4], a2[4][4];   // sums of the output row that ends next, and of the one after it
#pragma unroll
    for (int q = 0; q < 4; q++)
#pragma unroll
        for (int c = 0; c < 4; c++) { a1[q][c] = 0; a2[q][c] = 0; }
    int o[4][4];
    auto row = [&](int next, bool more) {   // one input row; next: the row to load
        uint32_t d[6];
#pragma unroll
        for (int i = 0; i < 6; i++) {
            const uint32_t m = cmask[i] & rmask;
            d[i] = decode4_lut<MODE>((nx[i] & m) | (p.zero4 & ~m), p.dx);
        }
        if (OUT || more) load_row(next, nx);
#pragma unroll
        for (int h = 0; h < 2; h++) {        // columns 2h .. 2h+3 serve outputs 2h and 2h+1
            const uint32_t x01 = __builtin_amdgcn_perm(d[2 * h + 1], d[2 * h], 0x05010400u);
            const uint32_t x23 = __builtin_amdgcn_perm(d[2 * h + 1], d[2 * h], 0x07030602u);
            const uint32_t y01 = __builtin_amdgcn_perm(d[2 * h + 3], d[2 * h + 2], 0x05010400u);
            const uint32_t y23 = __builtin_amdgcn_perm(d[2 * h + 3], d[2 * h + 2], 0x07030602u);
            const uint32_t ch[4] = {__builtin_amdgcn_perm(y01, x01, 0x05040100u),
                                    __builtin_amdgcn_perm(y01, x01, 0x07060302u),
                                    __builtin_amdgcn_perm(y23, x23, 0x05040100u),
                                    __builtin_amdgcn_perm(y23, x23, 0x07060302u)};
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const int q = 2 * h;
                o[q][c] = __builtin_amdgcn_sdot4((int)ch[c], (int)wlo[2][c], a1[q][c], false);
                a1[q][c] = __builtin_amdgcn_sdot4((int)ch[c], (int)wlo[1][c], a2[q][c], false);
                a2[q][c] = __builtin_amdgcn_sdot4((int)ch[c], (int)wlo[0][c], 0, false);
                o[q + 1][c] = __builtin_amdgcn_sdot4((int)ch[c], (int)whi[2][c], a1[q + 1][c], false);
                a1[q + 1][c] = __builtin_amdgcn_sdot4((int)ch[c], (int)whi[1][c], a2[q + 1][c], false);
                a2[q + 1][c] = __builtin_amdgcn_sdot4((int)ch[c], (int)whi[0][c], 0, false);
            }
        }
    };
    uint32_t amax = 0;
#pragma unroll 1
    for (int i = 0; i < 2; i++) row(r0 + 1 + i - g.ph, true);   // the rows above the last one
#pragma unroll 1
    for (int r = r0; r < r1; r++) {          // input row r + 2 - ph is the last one of output row r
        row(r + 3 - g.ph, r + 1 < r1);
        const int64_t ob = (((int64_t)n * g.P + r) * g.Q + q0) * C + c0;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int64_t oo = ob + (int64_t)q * C;
            const f32x4 v{s * (float)o[q][0], s * (float)o[q][1], s * (float)o[q][2],
                          s * (float)o[q][3]};
            if (OUT == 0) {
                if (q0 + q >= g.Q) break;
                if (p.acc) *(int4*)(p.acc + oo) = make_int4(o[q][0], o[q][1], o[q][2], o[q][3]);
                if (p.post.on) amax = max(amax, post_apply4(p.post, p.y, oo, c0, v, post_res4(p.post, oo), qa));
                else if (p.y) *(f32x4*)(p.y + oo) = v;
            } else {
                f32x4 z = v;
                if (p.post.on) {   // a = 1, b = 0: -0 becomes +0
#pragma unroll
                    for (int c = 0; c < 4; c++) {
                        z[c] = v[c] + 0.0f;
                        if (p.post.relu) z[c] = z[c] > 0.0f ? z[c] : 0.0f;
                        amax = max(amax, __float_as_uint(z[c]) & 0x7fffffffu);
                    }
                }
                if (OUT == 1) *(f32x4*)(p.y + oo) = z;
                else *(uint32_t*)(p.post.codes + oo) =
                         q_ok ? code4(z, qa, q_r, q_fast, p.post.pp) : p.post.pp.zero_code * 0x01010101u;
            }
        }
    }
    if (p.post.on) post_absmax_flush(p.post, amax);
}

// OUT of k_dw3 for these outputs.
static int dw3_out(const ConvGeom& g, const int32_t* acc, const float* y, const Post& P) {
    const bool lean = g.Q >= 4 && !acc && !P.a && !P.b && !P.res && (y != nullptr) != (P.codes != nullptr) &&
                      (uintptr_t)P.codes % 4 == 0;
    return !lean ? 0 : (y ? 1 : 2);
}

template <int MODE>
static void launch_dw3_mode(const Dw3Params& p, int out, int blocks, hipStream_t s) {
    if (out == 0) k_dw3<0, MODE><<<blocks, kDwThreads, 0, s>>>(p);
    else if (out == 1) k_dw3<1, MODE><<<blocks, kDwThreads, 0, s>>>(p);
    else k_dw3<2, MODE><<<blocks, kDwThreads, 0, s>>>(p);
}

static hipError_t launch_dw3(const ConvGeom& g, const uint8_t* x, const Fmt& fx, const float* alphaX,
                             const uint8_t* w, const Fmt& fw, const float* alphaW, int32_t* acc,
                             float* y, hipStream_t s, const Post* post) {
    Dw3Params p;
    p.g = g; p.x = x; p.w = w; p.alphaX = alphaX; p.alphaW = alphaW; p.acc = acc; p.y = y;
    p.dx = decode_info(fx);
    p.dw = decode_info(fw);
    p.zero4 = fx.zero_code * 0x01010101u;
    p.post = post ? *post : Post{};
    p.cols = (g.Q + 3) / 4;
    // strips as long as they leave 8 waves per CU (a strip rereads two rows): the tallest of
    // 16, 8, 4 and 2 rows that does
    const int64_t per_row = (int64_t)g.Nb * p.cols * (g.C / 4);
    const int64_t want = (int64_t)num_cus() * 8 * 64;
    p.rows = 16;
    while (p.rows > 2 && per_row * ((g.P + p.rows - 1) / p.rows) < want) p.rows /= 2;
    p.strips = (g.P + p.rows - 1) / p.rows;
    p.rows = (g.P + p.strips - 1) / p.strips;   // even strips
    p.strips = (g.P + p.rows - 1) / p.rows;
    p.total = (int)(per_row * p.strips);   // <= 2^30 + per_row: see dw3_fits
    const int blocks = (p.total + kDwThreads - 1) / kDwThreads;
    const int out = dw3_out(g, acc, y, p.post);
    if (p.dx.mode == 3) launch_dw3_mode<3>(p, out, blocks, s);
    else if (p.dx.mode == 4) launch_dw3_mode<4>(p, out, blocks, s);
    else launch_dw3_mode<5>(p, out, blocks, s);
    return hipGetLastError();
}

// The conditions of k_dw3: its byte permutes decode activations of at most five bits
// (longer formats would decode arithmetically, more work than the table kernels), and its
// dword loads and 16-byte stores need aligned tensors.  It walks a strip of rows per thread, a
// longer chain than one output's, and its general epilogue (OUT 0) is four times the code, while the
// other kernels copy the filter through LDS per workgroup: small calls with few channels are
// faster there.  Measured over 3800 shapes and forms (us, k_dwconv16 or k_dwconv / here):
//  * C % 16 == 0: the lean outputs and int32 sums are faster here at every size (16 channels
//    6.3 / 5.3, 960 10.4 / 4.5), the general ones from 64 channels on, 192 with an affine (affine
//    and codes at 14 x 14: 32 channels 8.1 / 9.4, 192 9.6 / 9.6, 960 14.2 / 9.4), or over 2^20 outputs;
//  * else: lean outputs with ReLU or max|z| (5.8 / 5.4), y from 16 channels, codes and sums
//    from 64, or over 2^18 (sums 2^19) outputs; other epilogues over 2^20 (affine and codes at 2^15
//    6.8 / 10.1, at 2^20 11.3 / 10.0);
//  * two or three columns, where threads are partly padding: C % 16 == 0 but for post-processing
//    of less than 48 channels in three columns (2 x 2, 32 channels, batch 8, sums 5.9 / 5.2; 3 x 3,
//    16 channels, affine and codes 9 % the other way); else large calls (100 channels at 3 x 3,
//    batch 512, sums 6.5 / 5.9);
//  * one column, three quarters padding: up to 3 x 10^5 outputs (codes 5 x 10^5: 144 channels, batch
//    4096, 7.1 / 8.0) of C % 16 == 0 or 96 channels, without post-processing of 64 to 144 channels
//    and more (batch 128, 96 channels, y 5.4 / 4.8; batch 1 5 % the other way).
static bool dw3_fits(const ConvGeom& g, const uint8_t* x, const Fmt& fx, const Fmt& fw,
                     const int32_t* acc, const float* y, const Post* post) {
    const Post P = post ? *post : Post{};
    const bool c16 = g.C % 16 == 0, affine = P.a || P.b;
    const int64_t outputs = (int64_t)g.Nb * g.P * g.Q * g.C;
    bool pays;
    if (dw3_out(g, acc, y, P)) pays = c16 || (P.on && y) || g.C >= (y ? 16 : 64) || outputs >= 1 << 18;
    else if (g.Q == 1 && P.on) pays = (c16 || g.C >= 96) && outputs < (c16 && P.codes ? 500000 : 300000);
    else if (g.Q == 1) pays = c16 && outputs < 300000 && (g.C >= 144 || (g.C >= 64 && outputs >= 3000));
    else if (g.Q < 4 && c16) pays = g.Q == 2 || !P.on || g.C >= 48;
    else if (g.Q < 4) pays = outputs >= (!P.on && g.C >= 64 ? 1 << 15 : (P.on && g.Q == 3 ? 1 << 20 : 1 << 19));
    else if (!P.on) pays = c16 || g.C >= 64 || outputs >= 1 << 19;
    else pays = (c16 && g.C >= (affine ? 192 : 64)) || outputs >= 1 << 20;
    return pays && g.R == 3 && g.S == 3 && g.sh == 1 && g.sw == 1 && g.C % 4 == 0 && fx.n <= 5 &&
           fx.max_int <= 127 && fw.max_int <= 127 && (uintptr_t)x % 4 == 0 &&
           (!acc || (uintptr_t)acc % 16 == 0) && (!y || (uintptr_t)y % 16 == 0) &&
           (int64_t)g.Nb * g.P * ((g.Q + 3) / 4) * (g.C / 4) < ((int64_t)1 << 30) &&
           (int64_t)g.W * g.C < ((int64_t)1 << 31);
}

hipError_t launch_dwconv(const ConvGeom& g, const uint8_t* x, const Fmt& fx, const float* alphaX,
                         const uint8_t* w, const Fmt& fw, const float* alphaW, int32_t* acc,
                         float* y, hipStream_t s, const Post* post) {
    if (dw3_fits(g, x, fx, fw, acc, y, post))
        return launch_dw3(g, x, fx, alphaX, w, fw, alphaW, acc, y, s, post);
    DwParams p;
    p.g = g; p.x = x; p.w = w; p.alphaX = alphaX; p.alphaW = alphaW; p.acc = acc; p.y = y;
    p.post = post ? *post : Post{};
    p.kx = fx.k; p.kw = fw.k;
    for (int c = 0; c < 256; c++) {
        p.tx[c] = (int16_t)decode_int(fx, (uint32_t)c);
        p.tw[c] = (int16_t)decode_int(fw, (uint32_t)c);
    }
    const bool vec = (g.C % 4 == 0) && ((uintptr_t)x % 4 == 0) && (!acc || (uintptr_t)acc % 16 == 0) &&
                     (!y || (uintptr_t)y % 16 == 0);
    if (g.C % 16 == 0 && g.C * g.R * g.S <= kDwMaxTaps && g.R * g.S <= kDw16MaxTaps &&
        (uintptr_t)x % 16 == 0 &&
        (!acc || (uintptr_t)acc % 16 == 0) && (!y || (uintptr_t)y % 16 == 0)) {
        const int CV = g.C / 16;
        const int64_t npix = (int64_t)g.Nb * g.P * g.Q;
        // blocks: a multiple of CV / gcd(CV, 256), so that the thread count is a multiple of CV
        int unit = CV;
        for (int d = 256; d > 1; d /= 2)
            if (unit % 2 == 0 && d > 1) unit /= 2; else break;
        int64_t want = (npix * CV + kDwThreads - 1) / kDwThreads;
        const int64_t cap = (int64_t)num_cus() * 4;
        if (want > cap) want = cap;
        int64_t blocks = (want + unit - 1) / unit * unit;
        if (blocks < unit) blocks = unit;
        const int pix_step = (int)(blocks * kDwThreads / CV);
        k_dwconv16<<<(int)blocks, kDwThreads, 0, s>>>(p, pix_step);
        return hipGetLastError();
    }
    const int64_t total = (int64_t)g.Nb * g.P * g.Q * (vec ? g.C / 4 : g.C);
    int64_t blocks = (total + kDwThreads - 1) / kDwThreads;
    // each block decodes the filters into LDS first: few blocks, each over many outputs
    const int64_t cap = (int64_t)num_cus() * 4;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    if (vec) k_dwconv<true><<<(int)blocks, kDwThreads, 0, s>>>(p);
    else k_dwconv<false><<<(int)blocks, kDwThreads, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace esb
