// Contraction over ESB codes (Sec. 4.2; multiplication eq. (15)) on int8 MFMA, gfx950.
//
// Codes are decoded to their exact integers m = q * 2^k while a tile moves from
// HBM to LDS: eq. (15) says a product of two ESB values is a (k+1)-bit by
// (k+1)-bit fraction product shifted by the exponents, so m_A * m_B is exactly
// 2^(kA+kB) * q_A * q_B and an integer dot product over m is exact.  When
// every |m| <= 127 the decoded tile feeds v_mfma_i32_16x16x64_i8 directly;
// otherwise each m is split as 256*hi + lo with int8 hi, lo, and the partial
// products are combined with weights 1, 256, 65536 (int32, wrap-around exact
// because the final sum fits int32).
//
// Tiles: BM x BN per workgroup (256 threads, 4 waves of WM x WN), BK = 64 bytes
// of reduction per step, LDS double buffer.  LDS rows are 64 bytes; the four
// 16-byte chunks of a row are XOR-swizzled by (row >> 1) & 3 so that the
// ds_read_b128 of 8 consecutive rows at one chunk covers all 32 banks.
// A is addressed as an implicit im2col of an NHWC tensor (a dense row-major
// matrix is the special case H = W = R = S = 1 with pixel pitch lda).
#include "esb_internal.h"

namespace esb {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int BK = 64;
constexpr int NT = 256;

struct GemmParams {
    int M, N, K;            // per-group GEMM sizes (K = R*S*Cg)
    ConvGeom ga;
    const uint8_t* A;
    const uint8_t* B;
    int64_t ldb;
    DecodeInfo da, db;
    const float* alphaA;
    const float* alphaB;
    int32_t* acc;
    float* y;
    int64_t ldc;
    uint32_t zeroA, zeroB;  // the +0 code of each operand (padding / out of range)
    Post post;              // fused post-processing of the outputs (post.on == 0: none)
};

// ------------------------------------------------------------------ decode
// Decoding through a 256-entry LDS table of (low byte | high byte << 8) per code, m = 256 * hi
// + lo with int8 hi, lo (hi is 0 and unused where every |m| <= 127): three operations and one
// LDS read per code for every format, where arithmetic takes about 20 and byte-permute tables
// branch on the format per dword (1000 x 1000 x 999: 28.7 us by permutes in ESB(5,2), 15.2
// by the table).
__device__ __forceinline__ uint16_t lut_entry(uint32_t c, const DecodeInfo& d) {
    const int m = decode_one(c, d);
    const int l = (int)(int8_t)(m & 0xff);
    return (uint16_t)(((uint32_t)l & 0xffu) | (((uint32_t)((m - l) >> 8) & 0xffu) << 8));
}
// Four codes to the high and low int8 planes.
__device__ __forceinline__ void decode4_table(uint32_t w, const uint16_t* lut, uint32_t& hi,
                                              uint32_t& lo) {
    const uint32_t p01 = (uint32_t)lut[w & 0xffu] | ((uint32_t)lut[(w >> 8) & 0xffu] << 16);
    const uint32_t p23 = (uint32_t)lut[(w >> 16) & 0xffu] | ((uint32_t)lut[w >> 24] << 16);
    lo = __builtin_amdgcn_perm(p23, p01, 0x06040200u);
    hi = __builtin_amdgcn_perm(p23, p01, 0x07050301u);
}

__device__ __forceinline__ int swz(int row, int chunk) {
    return row * BK + ((chunk ^ ((row >> 1) & 3)) << 4);
}

template <int P>
__device__ __forceinline__ void store_tile(int8_t* base, int plane_stride, int row, int chunk,
                                           uint4 codes, const uint16_t* lut) {
    const int off = swz(row, chunk);
    uint4 h = make_uint4(0u, 0u, 0u, 0u), l;
    decode4_table(codes.x, lut, h.x, l.x);
    decode4_table(codes.y, lut, h.y, l.y);
    decode4_table(codes.z, lut, h.z, l.z);
    decode4_table(codes.w, lut, h.w, l.w);
    *(uint4*)(base + off) = l;                                // plane 0: low
    if (P == 2) *(uint4*)(base + plane_stride + off) = h;     // plane 1: high
}

// ----------------------------------------------------------------- loaders
// A slot: one 16-byte chunk (row, chunk) of the BM x 64 tile, fixed per thread.
struct ASlot {
    int valid;     // row inside M
    int nimg, ih0, iw0;
    int r, s, cc;  // (r, s, c) of the chunk's first reduction index (VEC16 path)
};

__device__ __forceinline__ void a_slot_init(ASlot& sl, const GemmParams& g, int m, int chunk) {
    const ConvGeom& c = g.ga;
    sl.valid = m < g.M;
    const int mm = sl.valid ? m : 0;
    const int pq = c.P * c.Q;
    sl.nimg = mm / pq;
    const int rem = mm - sl.nimg * pq;
    const int p = rem / c.Q, q = rem - (rem / c.Q) * c.Q;
    sl.ih0 = p * c.sh - c.ph;
    sl.iw0 = q * c.sw - c.pw;
    const int kk = 16 * chunk;
    const int cg = max(c.Cg, 1);
    const int rs = kk / cg;
    sl.cc = kk - rs * cg;
    sl.r = rs / c.S;
    sl.s = rs - sl.r * c.S;
}

// Requires Cg >= 16 (the 16-byte path is only chosen for K > 0 with Cg % 16 == 0).
__device__ __forceinline__ void a_slot_advance(ASlot& sl, const ConvGeom& c) {
    if (c.Cg <= 0) return;
    sl.cc += BK;
    while (sl.cc >= c.Cg) {
        sl.cc -= c.Cg;
        if (++sl.s == c.S) { sl.s = 0; ++sl.r; }
    }
}

// VEC16: C/groups % 16 == 0, pitch % 16 == 0, 16-byte aligned base.
__device__ __forceinline__ uint4 a_load16(const ASlot& sl, const GemmParams& g, int k_start,
                                          int goff) {
    const ConvGeom& c = g.ga;
    const uint32_t z4 = g.zeroA * 0x01010101u;
    uint4 v = make_uint4(z4, z4, z4, z4);
    if (sl.valid && k_start < g.K) {
        const int ih = sl.ih0 + sl.r, iw = sl.iw0 + sl.s;
        if (ih >= 0 && ih < c.H && iw >= 0 && iw < c.W) {
            const uint8_t* p = g.A + (((int64_t)sl.nimg * c.H + ih) * c.W + iw) * c.pitch + goff + sl.cc;
            v = *(const uint4*)p;
        }
    }
    return v;
}

// Byte path for any geometry.  With a table (kt != nullptr) the reduction index
// kk maps to {address offset from the pixel at (ih0, iw0), r << 16 | s}, built
// once per workgroup; without it (long reductions) the division chain is used.
constexpr int kKtabMax = 2048;

__device__ __forceinline__ uint4 a_load1(const ASlot& sl, const GemmParams& g, int k_start,
                                         int goff, const int2* kt) {
    const ConvGeom& c = g.ga;
    uint32_t w[4];
    const int64_t pix = (((int64_t)sl.nimg * c.H + sl.ih0) * c.W + sl.iw0) * c.pitch + goff;
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
        uint32_t acc = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
            const int kk = k_start + 4 * q4 + b;
            uint32_t code = g.zeroA;
            if (sl.valid && kk < g.K) {
                int r, s;
                int64_t off;
                if (kt) {
                    const int2 e = kt[kk];
                    off = e.x;
                    r = e.y >> 16;
                    s = e.y & 0xffff;
                } else {
                    const int rs = kk / c.Cg;
                    const int ch = kk - rs * c.Cg;
                    r = rs / c.S;
                    s = rs - r * c.S;
                    off = ((int64_t)r * c.W + s) * c.pitch + ch;
                }
                const int ih = sl.ih0 + r, iw = sl.iw0 + s;
                if ((unsigned)ih < (unsigned)c.H && (unsigned)iw < (unsigned)c.W) code = g.A[pix + off];
            }
            acc |= code << (8 * b);
        }
        w[q4] = acc;
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// Sixteen codes of a contiguous row at reduction index k, any alignment (K >= 16): one
// unaligned 16-byte load; past the row's end it is the load of the row's last 16 codes moved
// down, with +0 codes (z4) behind.
struct __attribute__((packed)) U4Any { uint32_t v[4]; };
struct __attribute__((packed)) U1Any { uint32_t v; };
__device__ __forceinline__ uint4 row_load16(const uint8_t* row, int k, int K, uint32_t z4) {
    if (k >= K) return make_uint4(z4, z4, z4, z4);
    const U4Any u = *(const U4Any*)(row + (k + 16 <= K ? k : K - 16));
    if (k + 16 <= K) return make_uint4(u.v[0], u.v[1], u.v[2], u.v[3]);
    const int rem = K - k, sh = 8 * (16 - rem);          // rem codes stay: 1 .. 15
    uint64_t lo = ((uint64_t)u.v[1] << 32) | u.v[0], hi = ((uint64_t)u.v[3] << 32) | u.v[2];
    if (sh < 64) {
        lo = (lo >> sh) | (hi << (64 - sh));
        hi >>= sh;
    } else {
        lo = hi >> (sh - 64);
        hi = 0;
    }
    const uint64_t z8 = ((uint64_t)z4 << 32) | z4, ones = ~0ull;
    const uint64_t ml = rem >= 8 ? 0ull : ones << (8 * rem);
    const uint64_t mh = rem <= 8 ? ones : ones << (8 * (rem - 8));
    lo = (lo & ~ml) | (z8 & ml);
    hi = (hi & ~mh) | (z8 & mh);
    return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}

// B: output-channel row n (within the group), chunk of 16 reduction indices.
template <int BV>   // 16: NK vector, 4: NK unaligned vector, 1: NK bytes
__device__ __forceinline__ uint4 b_load(const GemmParams& g, int n, int k_start, int64_t brow0) {
    const uint32_t z4 = g.zeroB * 0x01010101u;
    uint4 v = make_uint4(z4, z4, z4, z4);
    if (n >= g.N || k_start >= g.K) return v;
    const uint8_t* row = g.B + (brow0 + n) * g.ldb;
    if (BV == 16) return *(const uint4*)(row + k_start);
    if (BV == 4) return row_load16(row, k_start, g.K, z4);
    uint32_t w[4];
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
        uint32_t acc = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
            const int kk = k_start + 4 * q4 + b;
            acc |= (kk < g.K ? (uint32_t)row[kk] : g.zeroB) << (8 * b);
        }
        w[q4] = acc;
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// KN layout: a thread takes blocks of four columns n .. n + 3 by four reduction indices, one
// dword per reduction index, and turns them around with byte permutes when it stores them.
__device__ __forceinline__ uint4 b_load_kn(const GemmParams& g, int n, int k_start, int64_t brow0) {
    const uint32_t z4 = g.zeroB * 0x01010101u;
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const int kk = k_start + q;
        w[q] = z4;
        if (kk < g.K && n < g.N) {
            const uint8_t* p = g.B + (int64_t)kk * g.ldb + brow0 + n;
            if (n + 4 <= g.N) {
                w[q] = ((const U1Any*)p)->v;
            } else {
                for (int b = 0; b < g.N - n; b++)
                    w[q] = (w[q] & ~(0xffu << (8 * b))) | ((uint32_t)p[b] << (8 * b));
            }
        }
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}
template <int P>
__device__ __forceinline__ void store_tile_kn(int8_t* base, int plane_stride, int row, int k4, uint4 r,
                                              const uint16_t* lut) {
    const uint32_t a01 = __builtin_amdgcn_perm(r.y, r.x, 0x05010400u);
    const uint32_t b01 = __builtin_amdgcn_perm(r.w, r.z, 0x05010400u);
    const uint32_t a23 = __builtin_amdgcn_perm(r.y, r.x, 0x07030602u);
    const uint32_t b23 = __builtin_amdgcn_perm(r.w, r.z, 0x07030602u);
    const uint32_t col[4] = {__builtin_amdgcn_perm(b01, a01, 0x05040100u),
                             __builtin_amdgcn_perm(b01, a01, 0x07060302u),
                             __builtin_amdgcn_perm(b23, a23, 0x05040100u),
                             __builtin_amdgcn_perm(b23, a23, 0x07060302u)};
#pragma unroll
    for (int j = 0; j < 4; j++) {
        uint32_t h = 0, l;
        decode4_table(col[j], lut, h, l);
        const int off = swz(row + j, k4 >> 2) + 4 * (k4 & 3);
        *(uint32_t*)(base + off) = l;
        if (P == 2) *(uint32_t*)(base + plane_stride + off) = h;
    }
}

// ------------------------------------------------------------------ kernel
// POST: the fused post-processing epilogue (a separate instantiation, so that
// the plain kernel keeps its register budget).
template <int BM, int BN, int WM, int WN, int PA, int PB, int AV, int BV, bool POST>
__global__ __launch_bounds__(NT) void k_contract(GemmParams g) {
    static_assert((BM / WM) * (BN / WN) == NT / 64, "4 waves per workgroup");
    constexpr int CA = (BM * 4 + NT - 1) / NT;   // A chunks per thread per stage
    constexpr int CB = (BN * 4 + NT - 1) / NT;   // B chunks, or blocks of 4 x 4 codes (KN)
    constexpr int TI = WM / 16, TJ = WN / 16;
    constexpr int NACC = PA + PB - 1;
    __shared__ __align__(16) int8_t sA[2][PA][BM * BK];
    __shared__ __align__(16) int8_t sB[2][PB][BN * BK];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int grp = blockIdx.z;
    const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
    const int wr = (wave / (BN / WN)) * WM, wc = (wave % (BN / WN)) * WN;
    const int goffA = grp * g.ga.Cg;
    const int64_t brow0 = (int64_t)grp * g.N;

    // byte path: the reduction-index table (short reductions)
    __shared__ int2 s_ktab[AV == 1 ? kKtabMax : 1];
    const int2* ktab = nullptr;
    if (AV == 1 && g.K <= kKtabMax &&
        (int64_t)g.ga.R * g.ga.W * g.ga.pitch + g.ga.pitch < 0x7fffffff) {
        for (int kk = threadIdx.x; kk < g.K; kk += NT) {
            const int cg = max(g.ga.Cg, 1);
            const int rs = kk / cg;
            const int ch = kk - rs * cg;
            const int r = rs / g.ga.S, s = rs - r * g.ga.S;
            s_ktab[kk] = make_int2((r * g.ga.W + s) * g.ga.pitch + ch, (r << 16) | s);
        }
        __syncthreads();
        ktab = s_ktab;
    }
    __shared__ uint16_t s_lutA[256], s_lutB[256];
    s_lutA[tid] = lut_entry((uint32_t)tid, g.da);
    s_lutB[tid] = lut_entry((uint32_t)tid, g.db);
    __syncthreads();
    ASlot as[CA];
    const uint8_t* arow[CA];   // AV == 4: the slot's row of K contiguous codes
#pragma unroll
    for (int i = 0; i < CA; i++) {
        const int c = tid + i * NT;
        a_slot_init(as[i], g, m0 + c / 4, c % 4);
        if (c >= BM * 4) as[i].valid = 0;
        arow[i] = g.A;
        if (AV == 4 && as[i].valid)
            arow[i] += (((int64_t)as[i].nimg * g.ga.H + as[i].ih0) * g.ga.W + as[i].iw0) * g.ga.pitch + goffA;
    }

    v4i acc[NACC][TI][TJ];
#pragma unroll
    for (int a = 0; a < NACC; a++)
#pragma unroll
        for (int i = 0; i < TI; i++)
#pragma unroll
            for (int j = 0; j < TJ; j++) acc[a][i][j] = v4i{0, 0, 0, 0};

    uint4 ra[CA], rb[CB];
    auto load_stage = [&](int k0) {
#pragma unroll
        for (int i = 0; i < CA; i++) {
            const int c = tid + i * NT;
            const int kst = k0 + 16 * (c % 4);
            if (AV == 4)
                ra[i] = row_load16(arow[i], as[i].valid ? kst : g.K, g.K, g.zeroA * 0x01010101u);
            else
                ra[i] = (AV == 16) ? a_load16(as[i], g, kst, goffA) : a_load1(as[i], g, kst, goffA, ktab);
        }
#pragma unroll
        for (int i = 0; i < CB; i++) {
            const int c = tid + i * NT;
            if constexpr (BV == 2) {
                if (c < BN * 4) rb[i] = b_load_kn(g, n0 + 4 * (c % (BN / 4)), k0 + 4 * (c / (BN / 4)), brow0);
            } else {
                rb[i] = b_load<BV>(g, n0 + c / 4, k0 + 16 * (c % 4), brow0);
            }
        }
    };
    auto store_stage = [&](int buf) {
#pragma unroll
        for (int i = 0; i < CA; i++) {
            const int c = tid + i * NT;
            if (c < BM * 4) store_tile<PA>(&sA[buf][0][0], BM * BK, c / 4, c % 4, ra[i], s_lutA);
        }
#pragma unroll
        for (int i = 0; i < CB; i++) {
            const int c = tid + i * NT;
            if (c < BN * 4) {
                if constexpr (BV == 2)
                    store_tile_kn<PB>(&sB[buf][0][0], BN * BK, 4 * (c % (BN / 4)), c / (BN / 4), rb[i], s_lutB);
                else
                    store_tile<PB>(&sB[buf][0][0], BN * BK, c / 4, c % 4, rb[i], s_lutB);
            }
        }
    };
    auto advance = [&]() {
        if (AV == 16) {
#pragma unroll
            for (int i = 0; i < CA; i++) a_slot_advance(as[i], g.ga);
        }
    };

    const int KT = (g.K + BK - 1) / BK;
    load_stage(0);
    advance();
    store_stage(0);
    __syncthreads();
    for (int kt = 0; kt < KT; kt++) {
        const int buf = kt & 1;
        if (kt + 1 < KT) { load_stage((kt + 1) * BK); advance(); }
        v4i fa[PA][TI], fb[PB][TJ];
#pragma unroll
        for (int p = 0; p < PA; p++)
#pragma unroll
            for (int i = 0; i < TI; i++)
                fa[p][i] = *(const v4i*)&sA[buf][p][swz(wr + 16 * i + (lane & 15), lane >> 4)];
#pragma unroll
        for (int p = 0; p < PB; p++)
#pragma unroll
            for (int j = 0; j < TJ; j++)
                fb[p][j] = *(const v4i*)&sB[buf][p][swz(wc + 16 * j + (lane & 15), lane >> 4)];
#pragma unroll
        for (int i = 0; i < TI; i++)
#pragma unroll
            for (int j = 0; j < TJ; j++)
#pragma unroll
                for (int pa = 0; pa < PA; pa++)
#pragma unroll
                    for (int pb = 0; pb < PB; pb++)
                        acc[pa + pb][i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                            fa[pa][i], fb[pb][j], acc[pa + pb][i][j], 0, 0, 0);
        if (kt + 1 < KT) store_stage(buf ^ 1);
        __syncthreads();
    }

    // epilogue: lane holds rows 4*(lane>>4) + r, column lane & 15 of each 16x16 block
    float s = 0.0f;
    if (g.y || POST) s = ldexpf(g.alphaA[0] * g.alphaB[0], -(g.da.k + g.db.k));
    auto ival = [&](int i, int j, int r) {
        uint32_t v = (uint32_t)acc[0][i][j][r];
        if (NACC > 1) v += (uint32_t)acc[NACC > 1 ? 1 : 0][i][j][r] << 8;
        if (NACC > 2) v += (uint32_t)acc[NACC > 2 ? 2 : 0][i][j][r] << 16;
        return (int32_t)v;
    };
    if constexpr (POST) {
        // fused post-processing through LDS, one row of 16x16 blocks at a time: each
        // wave's 16 x WN slab of scaled values is read back four outputs per lane, so
        // the post-processing code stays outside the unrolled register loops
        static_assert(NT / 64 * 16 * WN * 4 <= sizeof(sA), "post slabs fit the A buffers");
        float* slab = (float*)&sA[0][0][0] + wave * 16 * WN;
        const float qa = post_alpha(g.post);
        uint32_t amax = 0;
#pragma unroll
        for (int i = 0; i < TI; i++) {
            __syncthreads();
#pragma unroll
            for (int j = 0; j < TJ; j++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const int rl = 4 * (lane >> 4) + r, cl = 16 * j + (lane & 15);
                    const int row = m0 + wr + 16 * i + rl, col = n0 + wc + cl;
                    const int32_t iv = ival(i, j, r);
                    if (g.acc && row < g.M && col < g.N)
                        g.acc[(int64_t)row * g.ldc + (int64_t)grp * g.N + col] = iv;
                    slab[rl * WN + cl] = s * (float)iv;
                }
            __syncthreads();
#pragma unroll 1
            for (int e = 4 * lane; e < 16 * WN; e += 256) {
                const int rl = e / WN, cl = e - rl * WN;
                const int row = m0 + wr + 16 * i + rl, col = n0 + wc + cl;
                if (row < g.M && col < g.N) {
                    const int64_t ch = (int64_t)grp * g.N + col;
                    amax = max(amax, post_store4(g.post, g.y, (int64_t)row * g.ldc + ch, ch,
                                                 *(const f32x4*)(slab + e), min(4, g.N - col), qa));
                }
            }
        }
        post_absmax_flush(g.post, amax);
        return;
    }
#pragma unroll
    for (int i = 0; i < TI; i++)
#pragma unroll
        for (int j = 0; j < TJ; j++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int row = m0 + wr + 16 * i + 4 * (lane >> 4) + r;
                const int col = n0 + wc + 16 * j + (lane & 15);
                if (row < g.M && col < g.N) {
                    const int32_t iv = ival(i, j, r);
                    const int64_t o = (int64_t)row * g.ldc + (int64_t)grp * g.N + col;
                    if (g.acc) g.acc[o] = iv;
                    if (g.y) g.y[o] = s * (float)iv;
                }
            }
}

// ------------------------------------------------------------------ launch
DecodeInfo decode_info(const Fmt& f) {
    DecodeInfo d;
    d.n = f.n;
    d.k = f.k;
    d.emax = f.N;
    d.split = f.max_int > 127;
    d.mode = d.split ? 0 : (f.n <= 3 ? 3 : (f.n == 4 ? 4 : (f.n == 5 ? 5 : 0)));
    for (int w = 0; w < 8; w++) {
        uint32_t v = 0;
        for (int b = 0; b < 4; b++) {
            const uint32_t c = (uint32_t)(4 * w + b) & ((1u << f.n) - 1u);
            const int m = d.split ? 0 : decode_int(f, c);
            v |= ((uint32_t)m & 0xffu) << (8 * b);
        }
        d.lut[w] = v;
    }
    return d;
}

template <int BM, int BN, int WM, int WN, int PA, int PB, int AV, int BV>
static void launch_t(const GemmParams& g, int groups, hipStream_t s) {
    dim3 grid((g.M + BM - 1) / BM, (g.N + BN - 1) / BN, groups);
    if (g.post.on) k_contract<BM, BN, WM, WN, PA, PB, AV, BV, true><<<grid, NT, 0, s>>>(g);
    else k_contract<BM, BN, WM, WN, PA, PB, AV, BV, false><<<grid, NT, 0, s>>>(g);
}

// Loader pairs: A by 16 aligned bytes, 16 unaligned ones of a contiguous row (4) or bytes (1);
// B the same or KN blocks (2).
template <int BM, int BN, int WM, int WN, int PA, int PB>
static void launch_loaders(const GemmParams& g, int groups, int av, int bv, hipStream_t s) {
    if (av == 16) {
        if (bv == 16) launch_t<BM, BN, WM, WN, PA, PB, 16, 16>(g, groups, s);
        else if (bv == 2) launch_t<BM, BN, WM, WN, PA, PB, 16, 2>(g, groups, s);
        else launch_t<BM, BN, WM, WN, PA, PB, 16, 4>(g, groups, s);   // K >= 16 here
    } else if (av == 4) {
        if (bv == 2) launch_t<BM, BN, WM, WN, PA, PB, 4, 2>(g, groups, s);
        else launch_t<BM, BN, WM, WN, PA, PB, 4, 4>(g, groups, s);
    } else {
        if (bv == 2) launch_t<BM, BN, WM, WN, PA, PB, 1, 2>(g, groups, s);
        else if (bv == 1) launch_t<BM, BN, WM, WN, PA, PB, 1, 1>(g, groups, s);
        else launch_t<BM, BN, WM, WN, PA, PB, 1, 4>(g, groups, s);
    }
}

hipError_t launch_contraction(int M, int N, int K, int groups, const ConvGeom& ga,
                              const uint8_t* A, const DecodeInfo& da, const float* alphaA,
                              const uint8_t* B, int64_t ldb, int b_layout, const DecodeInfo& db,
                              const float* alphaB, int32_t* acc, float* y, int64_t ldc,
                              int /*out_col_per_group*/, hipStream_t s, const Post* post) {
    if (M <= 0 || N <= 0) return hipSuccess;
    GemmParams g;
    g.M = M; g.N = N; g.K = K; g.ga = ga;
    g.A = A; g.B = B; g.ldb = ldb; g.da = da; g.db = db;
    g.alphaA = alphaA; g.alphaB = alphaB; g.acc = acc; g.y = y; g.ldc = ldc;
    g.post = post ? *post : Post{};
    g.zeroA = (uint32_t)da.emax << da.k;
    g.zeroB = (uint32_t)db.emax << db.k;
    const bool a16 = (K > 0) && (ga.Cg >= 16) && (ga.Cg % 16 == 0) && (ga.pitch % 16 == 0) &&
                     ((uintptr_t)A % 16 == 0) &&
                     ((int64_t)groups * ga.Cg <= ga.pitch);
    // Rows of at least 16 contiguous codes that are not aligned take unaligned 16-byte loads
    // (1000 x 1000 x 999 in ESB(5,2): 71.6 us by single bytes, 15.2 here, and in ESB(6,2) 73.8 and 16.6; KN by 4 x 4 blocks
    // 2000 x 3000 x 2048 165 -> 84); the byte path stays for convolutions with channels that
    // are no multiple of 16 and for shorter rows.
    int bv;
    if (b_layout == 1) bv = 2;
    else if (K < 16) bv = 1;
    else bv = (K % 16 == 0) && (ldb % 16 == 0) && ((uintptr_t)B % 16 == 0) ? 16 : 4;
    const bool rows = K >= 16 && ga.R == 1 && ga.S == 1 && ga.ph == 0 && ga.pw == 0;
    const int av = a16 ? 16 : (rows ? 4 : 1);
    if (da.split || db.split) {
        if (da.split && db.split) launch_loaders<64, 64, 32, 32, 2, 2>(g, groups, av, bv, s);
        else if (da.split) launch_loaders<64, 64, 32, 32, 2, 1>(g, groups, av, bv, s);
        else launch_loaders<64, 64, 32, 32, 1, 2>(g, groups, av, bv, s);
        return hipGetLastError();
    }
    // tile choice: the largest tile that still gives every CU a workgroup
    const int64_t cus = num_cus();
    auto tiles = [&](int bm, int bn) {
        return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * groups;
    };
    if (N > 64 && tiles(128, 128) >= cus) launch_loaders<128, 128, 64, 64, 1, 1>(g, groups, av, bv, s);
    else if (tiles(64, 64) >= cus) launch_loaders<64, 64, 32, 32, 1, 1>(g, groups, av, bv, s);
    else launch_loaders<64, 32, 32, 16, 1, 1>(g, groups, av, bv, s);
    return hipGetLastError();
}

}  // namespace esb
