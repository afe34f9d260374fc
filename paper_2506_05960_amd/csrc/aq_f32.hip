// fp32 decode path: layers whose tile dtype is fp32, where the matrix-core
// fp16/bf16 rounding of the weight tile is not wanted.  Weights are expanded
// from codes in fp32 (any group size g) and contracted with fp32 matrix-core
// products (v_mfma_f32_32x32x2_f32: exact fp32 operands, fp32 accumulation).
//
// Work split.  A workgroup owns 32 TM tokens x 32 output channels and its NW
// waves split K into contiguous runs, so that a small layer still puts many
// waves on the chip; the partial tiles meet in LDS and are added in wave
// order.  Each step of a wave covers 8 k: a lane loads 4 consecutive
// activations of each of its tokens and decodes 4 consecutive weights of its
// channel (half a group of g = 8: one 16-byte read per codeword), straight
// into operand registers, and four products per 32 tokens consume them.
//
// Bound by the vector-memory path of the few compute units a small layer
// occupies: a wave's 64 lanes read 32 different rows, so an instruction costs
// tens of cycles whatever it fetches (codes read byte by byte for every step
// and codebook took most of a 64 x 256 -> 256 layer's time).  So where M
// divides 16 and B <= 8, a lane reads the codes of 16 / M groups as one
// 16-byte piece of the table path's code layout, in which consecutive channels
// are consecutive, and gathers its codewords from a copy of the codebooks in
// LDS (about 50 cycles a gather, 130 through the L1).
//
// Measured, M = 2: 64 tokens x 256 -> 256 5.9 us (52.8 with the 64 x 64 vector-ALU
// tiles this replaces, which decoded 16 k at a time between barriers); 256 x
// 512 -> 512 7.5 us (101); 1000 x 704 -> 704 22.8 us (131), 43 TFLOP/s.
#include <algorithm>

#include "aq_device.h"

namespace aq {

constexpr int kF32Tile = 32;
constexpr int kF32Steps = 4;       // steps of 8 k whose loads are in flight together
constexpr int kF32Pitch = kF32Tile + 1;
constexpr int64_t kF32GridX = 1 << 20;

// MC > 0: g == 8 and M == MC, codes in chunks of 16 bytes and codebooks in LDS;
// else one of
constexpr int kF32AnyG = 0;    // any group size, codewords value by value from memory
constexpr int kF32G8 = -1;     // g == 8, any M and B, codewords from memory

template <int XT, typename CodeT, int MC, int NW, int TM>
__global__ void __launch_bounds__(64 * NW)
f32_fwd_kernel(Geom geo, const float* __restrict__ cb32, const CodeT* __restrict__ codes,
               const float* __restrict__ scales, const void* __restrict__ X, const float* __restrict__ x_scales,
               void* __restrict__ Y, int y_dtype, int tiles_n) {
    extern __shared__ __attribute__((aligned(16))) float lds_f32[];   // codebooks, then the partial tiles
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, q = lane >> 5;
    const unsigned tile = blockIdx.y * gridDim.x + blockIdx.x;
    const int64_t m0 = (int64_t)(tile / (unsigned)tiles_n) * (kF32Tile * TM);
    const int n0 = (int)(tile % (unsigned)tiles_n) * kF32Tile;
    if (m0 >= geo.tokens) return;              // past the last tile (the whole workgroup)
    const int g = geo.g, M = geo.M, K = geo.K;
    const int nk = 1 << geo.B;

    if constexpr (MC > 0) {
        const int n4 = MC * nk * 2;
        for (int i = tid; i < n4; i += 64 * NW)
            reinterpret_cast<floatx4*>(lds_f32)[i] = reinterpret_cast<const floatx4*>(cb32)[i];
    }
    // rows past the last token or channel repeat it; their outputs are not stored
    int64_t tok[TM];
#pragma unroll
    for (int a = 0; a < TM; ++a) {
        const int64_t t = m0 + 32 * a + l32;
        tok[a] = t < geo.tokens ? t : geo.tokens - 1;
    }
    const int co = min(n0 + l32, geo.C_out - 1);
    const CodeT* crow = codes + (int64_t)co * geo.G * M;
    const bool xvec = XT == AQ_F32 && !geo.conv && K % 4 == 0;   // whole 16-byte pieces of a row

    floatx16 acc[TM];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][r] = 0.0f;

    // a convolution's token: its image and the input position of kernel tap (0, 0)
    int64_t img[TM];
    int ih0[TM], iw0[TM];
#pragma unroll
    for (int a = 0; a < TM; ++a) {
        img[a] = 0;
        ih0[a] = iw0[a] = 0;
        if (geo.conv) {
            const int64_t plane = (int64_t)geo.OH * geo.OW, b = tok[a] / plane;
            const int p = (int)(tok[a] - b * plane), oh = p / geo.OW;
            img[a] = b * geo.cin * (int64_t)geo.H * geo.W;
            ih0[a] = oh * geo.stride - geo.pad;
            iw0[a] = (p - oh * geo.OW) * geo.stride - geo.pad;
        }
    }
    const int khw = geo.kh * geo.kw;
    auto load_x = [&](auto& xv, int u, int k) {   // k .. k + 3 of every token (past K: the last ones again)
        if (geo.conv) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int ke = min(k + e, K - 1);
                int c = ke, r = 0, s = 0;
                if (khw != 1) {
                    c = ke / khw;
                    r = (ke - c * khw) / geo.kw;
                    s = ke - c * khw - r * geo.kw;
                }
#pragma unroll
                for (int a = 0; a < TM; ++a) {
                    const int ih = ih0[a] + r, iw = iw0[a] + s;
                    const bool in = ih >= 0 && ih < geo.H && iw >= 0 && iw < geo.W;
                    const float v = load_as_f32<XT>(X, in ? img[a] + ((int64_t)c * geo.H + ih) * geo.W + iw : 0);
                    xv[a][u][e] = in ? v : 0.0f;
                }
            }
            return;
        }
#pragma unroll
        for (int a = 0; a < TM; ++a) {
            if (xvec) {
                xv[a][u] = *reinterpret_cast<const floatx4*>(static_cast<const float*>(X) + tok[a] * K + min(k, K - 4));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) xv[a][u][e] = load_as_f32<XT>(X, tok[a] * K + min(k + e, K - 1));
            }
        }
    };
    if constexpr (MC > 0) {
        constexpr int JC = 16 / MC;                  // groups (steps) per chunk
        const int nchunk = (geo.G + JC - 1) / JC;
        const int per = (nchunk + NW - 1) / NW;
        const int c_end = min(nchunk, (wave + 1) * per);
        const u32x4* cchunk = reinterpret_cast<const u32x4*>(codes) + co;
        u32x4 cw = {};
        if (wave * per < c_end) cw = cchunk[(int64_t)(wave * per) * geo.C_out];
        __syncthreads();
        for (int c = wave * per; c < c_end; ++c) {
            constexpr int U = JC < 8 ? JC : 8;       // steps whose operands are in registers together
            const u32x4 cur = cw;
            if (c + 1 < c_end) cw = cchunk[(int64_t)(c + 1) * geo.C_out];
#pragma unroll
            for (int h = 0; h < JC / U; ++h) {
                if (c * JC + h * U >= geo.G) break;   // a last chunk that ends before its second half
                floatx4 xv[TM][U], wv[U];
#pragma unroll
                for (int u = 0; u < U; ++u) load_x(xv, u, 8 * (c * JC + h * U + u) + 4 * q);
#pragma unroll
                for (int u = 0; u < U; ++u) {
#pragma unroll
                    for (int m = 0; m < MC; ++m) {
                        const int i = (h * U + u) * MC + m;
                        const uint32_t code = (cur[i >> 2] >> (8 * (i & 3))) & 0xFFu;
                        const floatx4 w = *reinterpret_cast<const floatx4*>(lds_f32 + (m * nk + code) * 8 + 4 * q);
#pragma unroll
                        for (int e = 0; e < 4; ++e) wv[u][e] = m == 0 ? w[e] : __fadd_rn(wv[u][e], w[e]);
                    }
                    if (c * JC + h * U + u >= geo.G) {   // past K (uniform): zeros
                        wv[u] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                        for (int a = 0; a < TM; ++a) xv[a][u] = wv[u];
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int a = 0; a < TM; ++a)
                            acc[a] = __builtin_amdgcn_mfma_f32_32x32x2f32(xv[a][u][e], wv[u][e], acc[a], 0, 0, 0);
            }
        }
    } else {
        const int nstep = (K + 7) / 8;
        const int per = (nstep + NW - 1) / NW;
        const int s_end = min(nstep, (wave + 1) * per);
        for (int s0 = wave * per; s0 < s_end; s0 += kF32Steps) {
            // steps past the wave's last read its last group (every address is
            // in range) and become zeros before the products
            floatx4 xv[TM][kF32Steps], wv[kF32Steps];
#pragma unroll
            for (int u = 0; u < kF32Steps; ++u) load_x(xv, u, 8 * (s0 + u) + 4 * q);
            if constexpr (MC == kF32G8) {
                const CodeT* cp[kF32Steps];
#pragma unroll
                for (int u = 0; u < kF32Steps; ++u) cp[u] = crow + (int64_t)min(s0 + u, s_end - 1) * M;
                for (int m = 0; m < M; ++m) {
                    int64_t row[kF32Steps];
#pragma unroll
                    for (int u = 0; u < kF32Steps; ++u) row[u] = (int64_t)m * nk + cp[u][m];
#pragma unroll
                    for (int u = 0; u < kF32Steps; ++u) {
                        const floatx4 c = *reinterpret_cast<const floatx4*>(cb32 + row[u] * 8 + 4 * q);
#pragma unroll
                        for (int e = 0; e < 4; ++e) wv[u][e] = m == 0 ? c[e] : __fadd_rn(wv[u][e], c[e]);
                    }
                }
            } else {
#pragma unroll
                for (int u = 0; u < kF32Steps; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int k = min(8 * (s0 + u) + 4 * q + e, K - 1);
                        const int j = k / g, t = k - j * g;
                        const CodeT* bp = crow + (int64_t)j * M;
                        float w = cb32[(int64_t)bp[0] * g + t];
                        for (int m = 1; m < M; ++m) w = __fadd_rn(w, cb32[((int64_t)m * nk + bp[m]) * g + t]);
                        wv[u][e] = w;
                    }
            }
#pragma unroll
            for (int u = 0; u < kF32Steps; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool live = s0 + u < s_end && 8 * (s0 + u) + 4 * q + e < K;
                    wv[u][e] = live ? wv[u][e] : 0.0f;
#pragma unroll
                    for (int a = 0; a < TM; ++a) xv[a][u][e] = live ? xv[a][u][e] : 0.0f;
                }
#pragma unroll
            for (int u = 0; u < kF32Steps; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int a = 0; a < TM; ++a)
                        acc[a] = __builtin_amdgcn_mfma_f32_32x32x2f32(xv[a][u][e], wv[u][e], acc[a], 0, 0, 0);
        }
    }

    // lane (l32, q) holds channel l32 of tokens 32 a + 8 (r / 4) + 4 q + r % 4
    constexpr int PART = kF32Tile * TM * kF32Pitch;
    float* red = lds_f32;
    if constexpr (MC > 0) __syncthreads();   // the last codebook reads
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            red[wave * PART + (32 * a + 8 * (r >> 2) + 4 * q + (r & 3)) * kF32Pitch + l32] = acc[a][r];
    __syncthreads();
    constexpr int ROWS = kF32Tile * TM;
    for (int e = tid; e < ROWS * kF32Tile; e += 64 * NW) {
        // consecutive lanes store along the output's fast dimension
        const int row = geo.conv ? e % ROWS : e / kF32Tile;
        const int col = geo.conv ? e / ROWS : e % kF32Tile;
        const int64_t t = m0 + row;
        const int c = n0 + col;
        if (t >= geo.tokens || c >= geo.C_out) continue;
        float v = red[row * kF32Pitch + col];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += red[w * PART + row * kF32Pitch + col];
        v *= scales[c];
        if (x_scales) v *= x_scales[t];
        const int64_t yi = y_index(geo, t, c);
        if (y_dtype == AQ_F32) static_cast<float*>(Y)[yi] = v;
        else static_cast<uint16_t*>(Y)[yi] = f32_to_f16(v);
    }
}

// Short reductions in many tiles (f32_tile_better): 64 x 64 tiles on the vector ALUs, 16 k of activations and
// of decoded weights at a time staged in LDS, 4 x 4 outputs a thread.  Bound by the staging's
// index arithmetic and loads; no prologue or partial tiles, which at K = 8 take three times its time.
constexpr int kF32BM = 64, kF32BN = 64, kF32BK = 16;

template <int XT, typename CodeT>
__global__ void __launch_bounds__(256)
f32_tile_kernel(Geom geo, const float* __restrict__ cb32, const CodeT* __restrict__ codes,
               const float* __restrict__ scales, const void* __restrict__ X, const float* __restrict__ x_scales,
               void* __restrict__ Y, int y_dtype) {
    __shared__ float xs[kF32BK][kF32BM + 4];
    __shared__ float wsh[kF32BK][kF32BN + 4];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int64_t m0 = (int64_t)blockIdx.x * kF32BM;
    const int n0 = blockIdx.y * kF32BN;
    const int g = geo.g, M = geo.M;
    const int64_t nk = (int64_t)1 << geo.B;
    float acc[4][4] = {};

    for (int k0 = 0; k0 < geo.K; k0 += kF32BK) {
        // 64 x 16 activations and 64 x 16 decoded weights, 4 of each per thread
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = tid + q * 256;
            const int row = e & 63;
            const int kk = e >> 6;
            const int k = k0 + kk;
            const int64_t tok = m0 + row;
            xs[kk][row] = (tok < geo.tokens && k < geo.K) ? x_elem<XT>(geo, X, tok, k) : 0.0f;
            const int co = n0 + row;
            float w = 0.0f;
            if (co < geo.C_out && k < geo.K) {
                const int j = k / g;
                const int t = k - j * g;
                const CodeT* bp = codes + ((int64_t)co * geo.G + j) * M;
                w = cb32[(int64_t)bp[0] * g + t];
                for (int m = 1; m < M; ++m) w = __fadd_rn(w, cb32[((int64_t)m * nk + bp[m]) * g + t]);
            }
            wsh[kk][row] = w;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kF32BK; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = xs[kk][ty * 4 + i];
                b[i] = wsh[kk][tx * 4 + i];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) acc[i][jj] = fmaf(a[i], b[jj], acc[i][jj]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t tok = m0 + ty * 4 + i;
        if (tok >= geo.tokens) continue;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int co = n0 + tx * 4 + jj;
            if (co >= geo.C_out) continue;
            float v = acc[i][jj] * scales[co];
            if (x_scales) v *= x_scales[tok];
            const int64_t yi = y_index(geo, tok, co);
            if (y_dtype == AQ_F32) static_cast<float*>(Y)[yi] = v;
            else static_cast<uint16_t*>(Y)[yi] = f32_to_f16(v);
        }
    }
}

template <int XT, typename CodeT, int MC, int NW, int TM>
static hipError_t f32_launch_cfg(const Geom& geo, const DeviceWeights& w, const void* X, const float* x_scales,
                                 void* Y, int y_dtype, hipStream_t st) {
    auto kern = f32_fwd_kernel<XT, CodeT, MC, NW, TM>;
    const int64_t tm = (geo.tokens + kF32Tile * TM - 1) / (kF32Tile * TM);
    const int tn = (geo.C_out + kF32Tile - 1) / kF32Tile;
    if (tm * tn >= (int64_t(1) << 31)) return hipErrorInvalidConfiguration;
    // a launch holds fewer than 2^32 threads along x: more tiles go along y
    const unsigned gx = (unsigned)std::min<int64_t>(tm * tn, kF32GridX), gy = (unsigned)((tm * tn + gx - 1) / gx);
    const size_t part = (size_t)NW * TM * kF32Tile * kF32Pitch * sizeof(float);
    const size_t lds = std::max(part, MC > 0 ? ((size_t)geo.M << geo.B) * 8 * sizeof(float) : size_t(0));
    const hipError_t e = ensure_dynamic_lds((const void*)kern, lds);
    if (e != hipSuccess) return e;
    const void* codes = MC > 0 ? static_cast<const void*>(w.codes_lut) : w.codes;
    kern<<<dim3(gx, gy), 64 * NW, lds, st>>>(geo, w.cb32, static_cast<const CodeT*>(codes), w.scales, X,
                                                    x_scales, Y, y_dtype, tn);
    note_launch(st, "f32_fwd_kernel", {XT, 8 * (int)sizeof(CodeT), MC, NW, TM});
    return hipGetLastError();
}

// Waves per tile and tile height: 32-token tiles while those leave compute
// units idle, with four waves where K is at most four chunks, else sixteen;
// else 64-token tiles, which decode half as often.
template <int XT, typename CodeT, int MC>
static hipError_t f32_launch_mode(const Geom& geo, const DeviceWeights& w, const void* X, const float* x_scales,
                                  void* Y, int y_dtype, hipStream_t st) {
    const int64_t tiles = ((geo.tokens + kF32Tile - 1) / kF32Tile) * ((geo.C_out + kF32Tile - 1) / kF32Tile);
    if (tiles > 256) return f32_launch_cfg<XT, CodeT, MC, 4, 2>(geo, w, X, x_scales, Y, y_dtype, st);
    if (geo.K * std::max(1, MC) <= 512) return f32_launch_cfg<XT, CodeT, MC, 4, 1>(geo, w, X, x_scales, Y, y_dtype, st);
    return f32_launch_cfg<XT, CodeT, MC, 16, 1>(geo, w, X, x_scales, Y, y_dtype, st);
}

// Short reductions in many 64 x 64 tiles: the tile kernel.  A chunk of codes covers 128 / M k, so
// a short K leaves waves of the other kernel without one, and its workgroups copy the codebooks and
// add their partial tiles for little work; group sizes other than 8 read their codewords there value by value.
// The limits are where both are even, from some 2000 layers (tile kernel and the other, us: 16511
// tokens 8 -> 3172, M = 2 107 and 353; 5393 tokens 72 -> 1097, M = 1 38 and 64; 4554 tokens 24 -> 338, M = 2
// 12.0 and 16.4; 1808 tokens 120 -> 1422, M = 1 32.5 and 33.0; 1x1 17712 tokens 280 -> 666, M = 1 272 and 312;
// g = 12, M = 4 9727 tokens 144 -> 252 71 and 108).
template <int XT>
static bool f32_tile_better(const Geom& geo, const DeviceWeights& w) {
    const int64_t tiles = ((geo.tokens + kF32BM - 1) / kF32BM) * ((geo.C_out + kF32BN - 1) / kF32BN);
    if (tiles < 128 || geo.tokens >= (int64_t(1) << 29) || geo.C_out > (1 << 21)) return false;   // (more than its grid takes)
    const bool chunks = XT == AQ_F32 && w.codes_lut && geo.B <= 8;       // the other kernel's chunked codes, g = 8
    const int size = tiles < 200 ? 0 : tiles < 256 ? 1 : tiles < 300 ? 2 : tiles < 800 ? 3 : 4;
    // longest K by tiles, from 128, 200, 256, 300 and 800 up
    static constexpr int m1[5] = {16, 16, 16, 136, 192}, m1_conv[5] = {72, 72, 100, 160, 400};
    static constexpr int m2[5] = {16, 16, 16, 40, 88}, m2_conv[5] = {16, 24, 72, 104, 192};
    static constexpr int m4[5] = {0, 0, 0, 16, 16}, m4_conv[5] = {0, 0, 0, 40, 40};
    static constexpr int any[5] = {16, 33, 33, 48, 72}, any_m1[5] = {16, 16, 16, 33, 152};
    static constexpr int groups_m1[5] = {0, 48, 48, 150, 300}, groups_m2[5] = {0, 48, 48, 300, 350}, groups[5] = {0, 48, 48, 200, 400};
    const int* limit = geo.g != 8               ? (geo.M == 1 ? groups_m1 : geo.M == 2 ? groups_m2 : groups)
                       : chunks && geo.M == 1   ? (geo.conv ? m1_conv : m1)
                       : chunks && geo.M == 2   ? (geo.conv ? m2_conv : m2)
                       : chunks && geo.M == 4   ? (geo.conv ? m4_conv : m4)
                       : geo.M == 1             ? any_m1
                                                : any;
    return geo.K <= limit[size] || (!geo.conv && geo.g == 8 && geo.M == 3 && geo.K <= 33);
}

template <int XT, typename CodeT>
static hipError_t f32_launch_x(const Geom& geo, const DeviceWeights& w, const void* X, const float* x_scales, void* Y,
                               int y_dtype, hipStream_t st) {
    if (f32_tile_better<XT>(geo, w)) {
        const dim3 grid((unsigned)((geo.tokens + kF32BM - 1) / kF32BM), (unsigned)((geo.C_out + kF32BN - 1) / kF32BN));
        f32_tile_kernel<XT, CodeT><<<grid, 256, 0, st>>>(geo, w.cb32, static_cast<const CodeT*>(w.codes), w.scales, X,
                                                         x_scales, Y, y_dtype);
        note_launch(st, "f32_tile_kernel", {XT, 8 * (int)sizeof(CodeT)});
        return hipGetLastError();
    }
    if (geo.g != 8) return f32_launch_mode<XT, CodeT, kF32AnyG>(geo, w, X, x_scales, Y, y_dtype, st);
    if constexpr (sizeof(CodeT) == 1 && XT == AQ_F32) {
        // chunks of 16 code bytes per channel (the table path's code layout for these M:
        // its chunk of 16 / M groups fills 64 KB of table, so it never takes more)
        if (w.codes_lut && geo.M == 1) return f32_launch_mode<XT, CodeT, 1>(geo, w, X, x_scales, Y, y_dtype, st);
        if (w.codes_lut && geo.M == 2) return f32_launch_mode<XT, CodeT, 2>(geo, w, X, x_scales, Y, y_dtype, st);
        if (w.codes_lut && geo.M == 4) return f32_launch_mode<XT, CodeT, 4>(geo, w, X, x_scales, Y, y_dtype, st);
    }
    return f32_launch_mode<XT, CodeT, kF32G8>(geo, w, X, x_scales, Y, y_dtype, st);
}

template <typename CodeT>
static hipError_t f32_launch_codes(const Geom& geo, const DeviceWeights& w, const void* X, int x_dtype,
                                   const float* x_scales, void* Y, int y_dtype, hipStream_t st) {
    switch (x_dtype) {
    case AQ_F32: return f32_launch_x<AQ_F32, CodeT>(geo, w, X, x_scales, Y, y_dtype, st);
    case AQ_F16: return f32_launch_x<AQ_F16, CodeT>(geo, w, X, x_scales, Y, y_dtype, st);
    case AQ_BF16: return f32_launch_x<AQ_BF16, CodeT>(geo, w, X, x_scales, Y, y_dtype, st);
    default: return f32_launch_x<AQ_I8, CodeT>(geo, w, X, x_scales, Y, y_dtype, st);
    }
}

hipError_t launch_f32_forward(const Geom& geo, const DeviceWeights& w, const void* X, int x_dtype,
                              const float* x_scales, void* Y, int y_dtype, hipStream_t stream) {
    if (geo.B <= 8) return f32_launch_codes<uint8_t>(geo, w, X, x_dtype, x_scales, Y, y_dtype, stream);
    return f32_launch_codes<uint16_t>(geo, w, X, x_dtype, x_scales, Y, y_dtype, stream);
}

}  // namespace aq
