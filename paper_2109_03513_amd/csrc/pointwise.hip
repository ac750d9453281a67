// Contractions with a short reduction and many rows (pointwise convolutions, GEMMs of the
// same shape) on the fp8 MFMA of gfx950: K <= 256, any channel count, K a multiple of 8.
//
// Few operations per byte: what counts is that every code is loaded once, straight into the
// register layout of the matrix instructions, and that the outputs leave in wide stores.
// The tiled kernels stage 128 rows of operands through LDS for one or two 64-byte steps of
// reduction and spend their time on the set-up; where K is no multiple of 16 the general
// kernel even gathers single bytes.  Here
//  * the filter rows of a workgroup's channels are decoded to E4M3 once into LDS, rows of
//    64 KS + 16 bytes (an odd number of 16-byte groups: fragment reads without conflicts),
//    padded with zeros, so that whatever the pixel side holds past K adds nothing (decoded
//    codes are always finite in the formats admitted);
//  * a wave takes 32 pixels: lane (pixel, half) loads its own 32 bytes of every 64-byte step
//    in pieces of V = 16 or 8 bytes and decodes them in registers; the next tile's codes are
//    requested before this tile's outputs are written;
//  * the filter is the first matrix operand, so a lane ends up with four consecutive
//    channels of one pixel per four registers: 16-byte fp32 stores without a trip through
//    LDS; for codes, two lane-half swaps give every lane 16 consecutive channels of one pixel
//    and one 16-byte store.
// Exact under the admission rule of the other fp8 kernels (products at most 2^12, K times the
// largest product below 2^24): results equal theirs bit for bit.
// Measured at batch 32 and 56 x 56 (us, the path before and this one): 24 -> 144 channels
// codes out 84.5 / 19.4 (14.5 M codes: VALU of the scaling and coding), fp32 out 34.4 / 17.3
// (60 MB: HBM); 144 -> 24 fp32 out 15.6 / 8.9; one 28 x 28 image 24 -> 144 6.6 / 3.7.
#include "esb_internal.h"

namespace esb {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kPwThreads = 256;
constexpr int kPwLds = 60 * 1024;   // most of a workgroup's filter copy: two workgroups per CU

struct PwParams {
    const uint8_t* x;
    const uint8_t* w;
    const float* alphaX;
    const float* alphaW;
    int32_t* acc;
    float* y;
    int64_t pitch, ldw, ldc;   // bytes per input row (pixel), per filter row; outputs per row
    MmaDecode dx, dw;
    Post post;
    int M, N, K;
    int dense;                 // row m of the input at m pitch, else a strided pixel
    int H, W, P, Q, sh, sw;
    int nch;                   // channels per workgroup (multiple of 32)
    int tiles;                 // 32-row tiles
    int out_shift, kX, kW;
};

// V bytes of codes as V / 4 dwords.
template <int V>
__device__ __forceinline__ void pw_load(const uint8_t* p, uint32_t* d) {
    if (V == 16) {
        const uint4 v = *(const uint4*)p;
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    } else {
        const uint2 v = *(const uint2*)p;
        d[0] = v.x; d[1] = v.y;
    }
}

// OUT 0: every epilogue; OUT 1: fp32 outputs without affine (residual, ReLU and
// max|z| allowed), N and ldc multiples of 4, 16-byte aligned; OUT 2: codes without a residual
// either, N and ldc multiples of 16; OUT 3: int32 sums and perhaps plain fp32 outputs, aligned
// as for OUT 1 (16-byte stores: by single words, 4 channels of 32 pixels a wave, they took
// 1.5 to 4 times as long: 12544 x 1024 x 64 sums alone 41 us, here 16).
template <int KS, int OUT, int V>
__global__ __launch_bounds__(kPwThreads) void k_pw(PwParams p) {
    extern __shared__ __align__(16) uint8_t wl[];
    constexpr int RST = 64 * KS + 16;
    constexpr int PC = 32 / V, DW = V / 4;       // pieces per 32 bytes, dwords per piece
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lg = lane >> 5;
    const int wave = tid >> 6;
    const int n0 = blockIdx.y * p.nch, ncur = min(p.nch, p.N - n0);
    const int nb = (ncur + 31) / 32;

    // codes of a tile: row 32 tile + lr (rows past M repeat the last one), step ks, bytes
    // 32 lg .. + 31 (pieces past K repeat the row's first: the filter is zero there)
    uint32_t raw[KS][8];
    auto fetch = [&](int tile) {
        const int m = min(32 * tile + lr, p.M - 1);
        const uint8_t* row;
        if (p.dense) {
            row = p.x + (int64_t)m * p.pitch;
        } else {
            const int pq = p.P * p.Q, n = m / pq, rem = m - n * pq, pp = rem / p.Q, q = rem - pp * p.Q;
            row = p.x + (((int64_t)n * p.H + pp * p.sh) * p.W + q * p.sw) * p.pitch;
        }
#pragma unroll
        for (int ks = 0; ks < KS; ks++)
#pragma unroll
            for (int j = 0; j < PC; j++) {
                const int off = 64 * ks + 32 * lg + V * j;
                pw_load<V>(row + (off < p.K ? off : 0), &raw[ks][DW * j]);
            }
    };
    int tile = blockIdx.x * 4 + wave;
    if (tile < p.tiles) fetch(tile);

    // the filter, four pieces in flight per thread
    {
        constexpr int PR = 64 * KS / V;          // pieces per row
        const int total = 32 * nb * PR;
        for (int i0 = tid; i0 < total; i0 += 4 * kPwThreads) {
            uint32_t d[4][DW];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int i = i0 + u * kPwThreads, r = i / PR, o = V * (i - r * PR);
                const bool in = i < total && r < ncur && o < p.K;
                pw_load<V>(p.w + (in ? (int64_t)(n0 + r) * p.ldw + o : 0), d[u]);
#pragma unroll
                for (int e = 0; e < DW; e++) d[u][e] = in ? dec_f8(d[u][e], p.dw) : 0u;
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int i = i0 + u * kPwThreads, r = i / PR, o = V * (i - r * PR);
                if (i < total) {
#pragma unroll
                    for (int e = 0; e < DW; e++) *(uint32_t*)(wl + r * RST + o + 4 * e) = d[u][e];
                }
            }
        }
    }
    float s = 0.0f;
    if (p.y || p.post.on) s = ldexpf(p.alphaX[0] * p.alphaW[0], -(p.kX + p.kW));
    const float qa = p.post.on ? post_alpha(p.post) : 0.0f;
    const bool q_ok = alpha_valid(qa), q_fast = fast_scale(qa);
    const float q_r = 1.0f / qa;
    uint32_t amax = 0;
    __syncthreads();

    for (; tile < p.tiles; tile += 4 * gridDim.x) {
        const int m = 32 * tile + lr;
        v8i xf[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ks++)
#pragma unroll
            for (int e = 0; e < 8; e++) xf[ks][e] = (int)dec_f8(raw[ks][e], p.dx);
        if (tile + 4 * (int)gridDim.x < p.tiles) fetch(tile + 4 * gridDim.x);
        // the residual of this lane's outputs, one channel block ahead
        f32x4 rnx[4];
        auto fetch_res = [&](int mm, int b) {
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const int cl = 32 * b + 8 * g + 4 * lg;
                rnx[g] = *(const f32x4*)(p.post.res + (int64_t)min(mm, p.M - 1) * p.ldc + n0 +
                                         (cl < ncur ? cl : 0));
            }
        };
        if (OUT == 1 && p.post.res) fetch_res(m, 0);
#pragma unroll 1
        for (int b = 0; b < nb; b++) {
            f32x4 res[4];
            if (OUT == 1 && p.post.res) {
#pragma unroll
                for (int g = 0; g < 4; g++) res[g] = rnx[g];
                if (b + 1 < nb) fetch_res(m, b + 1);
            }
            v16f a;
#pragma unroll
            for (int r = 0; r < 16; r++) a[r] = 0.0f;
            const uint8_t* wb = wl + (32 * b + lr) * RST + 32 * lg;
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
                const v4i lo = *(const v4i*)(wb + 64 * ks), hi = *(const v4i*)(wb + 64 * ks + 16);
                const v8i wf{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                a = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wf, xf[ks], a, 0, 0, 0, 127, 0, 127);
            }
            // register r: channel n0 + 32 b + 8 (r / 4) + 4 lg + r % 4 of pixel m
            if (OUT == 2) {
                uint32_t c[4];
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    f32x4 z;
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        z[e] = s * ldexpf(a[4 * g + e], p.out_shift) + 0.0f;   // a = 1, b = 0
                        if (p.post.relu) z[e] = z[e] > 0.0f ? z[e] : 0.0f;
                        // rows past M repeat row M - 1: the maximum may count them twice
                        if (p.post.absmax && 32 * b + 8 * g + 4 * lg < ncur)
                            amax = max(amax, __float_as_uint(z[e]) & 0x7fffffffu);
                    }
                    c[g] = q_ok ? code4(z, qa, q_r, q_fast, p.post.pp) : p.post.pp.zero_code * 0x01010101u;
                }
                // swap the upper lane half of the first with the lower half of the second
                const u32x2 s02 = __builtin_amdgcn_permlane32_swap(c[0], c[2], false, false);
                const u32x2 s13 = __builtin_amdgcn_permlane32_swap(c[1], c[3], false, false);
                const int ch = 32 * b + 16 * lg;
                if (m < p.M && ch < ncur)
                    *(uint4*)(p.post.codes + (int64_t)m * p.ldc + n0 + ch) =
                        make_uint4(s02[0], s02[1], s13[0], s13[1]);
            } else {
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    const int cl = 32 * b + 8 * g + 4 * lg, ch = n0 + cl;
                    const int64_t o = (int64_t)m * p.ldc + ch;
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; e++) v[e] = s * ldexpf(a[4 * g + e], p.out_shift);
                    if (m >= p.M || cl >= ncur) continue;
                    if (OUT == 3) {
                        v4i n;
#pragma unroll
                        for (int e = 0; e < 4; e++) n[e] = (int32_t)ldexpf(a[4 * g + e], p.out_shift);
                        *(v4i*)(p.acc + o) = n;
                        if (p.y) *(f32x4*)(p.y + o) = v;
                    } else if (OUT == 1) {
                        if (p.post.on) {
#pragma unroll
                            for (int e = 0; e < 4; e++) {
                                v[e] = v[e] + 0.0f;   // a = 1, b = 0
                                if (p.post.res) v[e] = v[e] + res[g][e];
                                if (p.post.relu) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
                                amax = max(amax, __float_as_uint(v[e]) & 0x7fffffffu);
                            }
                        }
                        *(f32x4*)(p.y + o) = v;
                    } else {
                        const int nv = min(4, ncur - cl);
                        if (p.acc) {
#pragma unroll
                            for (int e = 0; e < 4; e++)
                                if (e < nv) p.acc[o + e] = (int32_t)ldexpf(a[4 * g + e], p.out_shift);
                        }
                        if (p.post.on) {
                            amax = max(amax, post_store4(p.post, p.y, o, ch, v, nv, qa));
                        } else if (p.y) {
#pragma unroll
                            for (int e = 0; e < 4; e++)
                                if (e < nv) p.y[o + e] = v[e];
                        }
                    }
                }
            }
        }
    }
    if (p.post.on) post_absmax_flush(p.post, amax);
}

template <int KS, int V>
void launch_pw_t(const PwParams& p, int out, dim3 grid, size_t lds, hipStream_t s) {
    if (out == 0) k_pw<KS, 0, V><<<grid, kPwThreads, lds, s>>>(p);
    else if (out == 1) k_pw<KS, 1, V><<<grid, kPwThreads, lds, s>>>(p);
    else if (out == 2) k_pw<KS, 2, V><<<grid, kPwThreads, lds, s>>>(p);
    else k_pw<KS, 3, V><<<grid, kPwThreads, lds, s>>>(p);
}

int pw_vec(const ConvGeom& g, const uint8_t* x, const uint8_t* w, int64_t ldw, int K) {
    for (int v = 16; v >= 8; v >>= 1)
        if (K % v == 0 && g.pitch % v == 0 && ldw % v == 0 && (uintptr_t)x % v == 0 &&
            (uintptr_t)w % v == 0)
            return v;
    return 0;
}

// The instance for these outputs (OUT of k_pw).
int pw_out(int N, const int32_t* acc, const float* y, int64_t ldc, const Post& P) {
    const bool al4 = N % 4 == 0 && ldc % 4 == 0 && (uintptr_t)acc % 16 == 0 && (uintptr_t)y % 16 == 0 &&
                     (uintptr_t)P.res % 16 == 0;
    if (acc) return al4 && !P.on ? 3 : 0;
    if (P.a || P.b) return 0;
    if (y && !P.codes && al4) return 1;
    if (!y && !P.res && P.codes && N % 16 == 0 && ldc % 16 == 0 && (uintptr_t)P.codes % 16 == 0) return 2;
    return 0;
}

// Where the general instance (outputs in single words, post-processing per lane and channel)
// beats the tiled and general kernels, measured over 5000 shapes and forms (us, there / here):
// up to 16 channels, of which those pad a tile to 32 or 64 (64 -> 8 over 200704 rows, y
// and codes 36 / 10); few bytes per row, which those load singly or half empty (24 -> 99 over
// 200704 rows, codes 109 / 34); post-processing of channels in no multiple of four, which
// those also store in single words; codes alone over many rows.  Against it: single-word y
// or int32 stores in quantity (64 -> 1001 over 6272 rows, y, 11 / 26), and calls of a few
// rows, where its epilogue's instruction fetches count (one row, 64 -> 64, affine and codes 4.6 / 6.0).
bool pw_general(int M, int N, int K, const int32_t* acc, const float* y, const Post& P) {
    const bool al = K % 16 == 0;                 // rows the tiled kernels take
    const int64_t MN = (int64_t)M * N;
    if (!P.on) {
        if (N <= 16) return M >= 32 || !al;
        return K < 16 && MN < (acc && y ? 50000 : 600000);
    }
    if (acc) return N <= 16;
    if (M < 8) return K < 16 || N <= 8 || (!al && K >= 64 && N <= 16);
    if (N < 32) return true;
    if (P.codes && y) {
        const bool half = N > 32 && N <= 64 && K >= 16;    // a 64-channel tile, at least half full
        if (M >= 50000 && ((N <= 160 && N % 64 && !al && !half) || (N <= 64 && N % 4 && (al || !half)))) return true;
        if (K < 16) return MN < 3000000 || (M < 20000 && MN >= 6000000);
        if (N % 4) return MN >= 2048 && MN < 5600000;
        return N <= 44 && M >= 18000;
    }
    if (K < 16) return true;
    if (N % 4) {
        if (!y) return true;
        if (N < 44 && al && K >= 128 && M < 50000) return false;   // half of 64 channels is padding
        return N <= 256 || (P.res ? MN < 2000000 : K <= 224);
    }
    if (M >= 20000 && (K <= 224 || (N <= 64 && M >= 80000))) return true;
    if (!al) return MN >= 1000000;
    if (K <= 128 && N >= 256) return MN >= 3000000;
    return (MN >= 25000000 && N >= 256) || (N <= 32 && M >= 45000);
}

}  // namespace

bool pw_fits(const ConvGeom& g, int M, int N, int groups, const uint8_t* x, const Fmt& fx,
             const uint8_t* w, int64_t ldw, const Fmt& fw, const int32_t* acc, const float* y,
             int64_t ldc, const Post* post) {
    const int K = g.Cg;
    if (groups != 1 || g.R != 1 || g.S != 1 || g.ph != 0 || g.pw != 0 || K < 8 || K > 256 || N > 1024) return false;
    if (!mma_e4m3_ok(fx, fw, K) || pw_vec(g, x, w, ldw, K) == 0) return false;
    const Post P = post ? *post : Post{};
    const int out = pw_out(N, acc, y, ldc, P);
    const int64_t MN = (int64_t)M * N;
    if (out == 2) return true;
    // The tiled kernels stay for many fp32 or int32 outputs of 65 to 512 channels over aligned
    // reductions of at least 64: their 128-channel rows leave in longer runs (64 -> 128 over
    // 50176 pixels 10.4 us there, 10.9 here, with a residual 15.2 against 16.4; 128 -> 256
    // likewise 18.6 against 20.4), and for more channels over the longest reductions, whose filter
    // copies fill the LDS in several shares (256 -> 768 over 12544 pixels 17.8 against 22.2; with
    // ReLU from more outputs, 224 -> 1000 over 4704 14.7 against 12.6, over 6272 15.3 against 17.4).
    // Few rows, few channels and codes are faster here (64 -> 64 over 200704 24.2 against 16.1,
    // codes 37.7 against 14.3; 64 -> 256 over 3136 5.1 against 4.2).
    if (!P.codes && K % 16 == 0 && K >= 64 && (int64_t)M * K >= 600000) {
        if (N > 64 && N <= 512) return false;
        const bool relu = P.on && !P.res;
        if (N > 512 && K > 192 && M < 20000 && MN >= (relu ? 5800000 : 4000000) && MN < 15000000) return false;
    }
    if (out == 0) return pw_general(M, N, K, acc, y, P);
    // Output rows 4 KB apart, 32 of which a store instruction meets, share few of the memory
    // channels (8 -> 1024 over 50176 pixels 53 us there, 90 here, over 18816 25.4 and 31.1; 128 ->
    // 1024 over 18816 35.2 and 31.0, over 37632 51.6 and 57.5); with the
    // post-processing those kernels are slower too.
    if (!P.on && ldc % 1024 == 0 && MN >= (K < 64 ? 19000000 : 20000000) && K <= 192) return false;
    // Two output streams at once (64 -> 1024 over 12544 pixels 21.7 there, 34.1 here).
    return !(out == 3 && y && N > 64 && MN >= 3000000);
}

hipError_t launch_pw(const ConvGeom& g, int M, int N, const uint8_t* x, const Fmt& fx,
                     const float* alphaX, const uint8_t* w, int64_t ldw, const Fmt& fw,
                     const float* alphaW, int32_t* acc, float* y, int64_t ldc, hipStream_t s,
                     const Post* post) {
    PwParams p{};
    p.x = x; p.w = w; p.alphaX = alphaX; p.alphaW = alphaW; p.acc = acc; p.y = y;
    p.pitch = g.pitch; p.ldw = ldw; p.ldc = ldc;
    p.dx = mma_decode(fx, 1);
    p.dw = mma_decode(fw, 1);
    if (post) p.post = *post;
    p.M = M; p.N = N; p.K = g.Cg;
    p.dense = (g.H == 1 && g.W == 1) || (g.sh == 1 && g.sw == 1);
    p.H = g.H; p.W = g.W; p.P = g.P; p.Q = g.Q; p.sh = g.sh; p.sw = g.sw;
    p.out_shift = fx.k + fw.k + 12;
    p.kX = fx.k; p.kW = fw.k;
    const int V = pw_vec(g, x, w, ldw, p.K);
    const int KS = (p.K + 63) / 64;
    const int out = pw_out(N, acc, y, ldc, p.post);
    p.tiles = (int)(((int64_t)M + 31) / 32);
    // channels per workgroup: even shares of whole 32-channel blocks that fit the LDS, and
    // more shares (each decodes the rows again) where one wave per tile leaves fewer than 8
    // waves per CU: 128 -> 256 channels over 12544 pixels, codes out, 22.3 us in one share,
    // 11.8 in six (with 16 waves per CU as the aim other shapes lose: 256 -> 256 over 12544
    // 9.3 -> 12.7 us).  Up to 64 channels the number
    // of shares is rounded: a second one for the last third of the 8 waves costs more than it
    // gives (192 -> 64 over 65000 pixels 12.0 us in two, 9.4 in one); down for fp32 outputs over
    // the longest rows (256 -> 64 over 43000 11.8 and 9.4).
    const int blocks32 = (N + 31) / 32, most = kPwLds / (32 * (64 * KS + 16));
    int ny = (blocks32 + most - 1) / most;
    const int up = N > 64 ? p.tiles - 1 : (KS == 4 && out != 2 ? 0 : p.tiles / 2);
    const int want = (8 * num_cus() + up) / p.tiles;
    if (ny < want) ny = want < blocks32 ? want : blocks32;
    p.nch = 32 * ((blocks32 + ny - 1) / ny);
    const int gy = (N + p.nch - 1) / p.nch;
    const size_t lds = (size_t)p.nch * (64 * KS + 16);
    int64_t gx = (p.tiles + 3) / 4;
    const int64_t cap = ((int64_t)num_cus() * 4 + gy - 1) / gy;
    if (gx > cap) gx = cap;
    const dim3 grid((unsigned)gx, (unsigned)gy);
#define ESB_PW(KSV) case KSV: if (V == 16) launch_pw_t<KSV, 16>(p, out, grid, lds, s); \
                              else launch_pw_t<KSV, 8>(p, out, grid, lds, s); break;
    switch (KS) { ESB_PW(1) ESB_PW(2) ESB_PW(3) ESB_PW(4) default: return hipErrorInvalidValue; }
#undef ESB_PW
    return hipGetLastError();
}

}  // namespace esb
