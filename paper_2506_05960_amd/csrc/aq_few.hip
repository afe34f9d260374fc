// Forward of a linear-layer-shaped product for one to four tokens, gfx950:
// y[n][i] = s[i] * sum_j sum_m <x_n[j], C_m[b[i][j][m]]> with the codewords read
// straight from LDS (fp16 codebooks, g = 8, M in {1, 2, 4}, B <= 8, fp16 or int8
// input; eq. (4) with the sums exchanged as in the appendix, but without its
// table: at a handful of tokens a table entry is used too rarely to repay its
// dot product).
//
// Work split.  A workgroup owns R output rows and its eight waves cover all of
// K: a lane is (row l % R, one of the wave's 64 / R chunks) and takes every
// 512 / R-th chunk of 16 code bytes (16 / M groups, the table path's code
// layout).  R is 4 where C_out needs the workgroups, 8 or 16 where it fills the
// chip with fewer, which then copy X and the codebooks fewer times.
// Nothing is shared between workgroups, so one launch does it, where the table
// path needs a second one to add the partial sums of its chunk groups.  Every
// workgroup copies the codebooks (4 KB each) and all of X (fp16, int8 widened
// exactly) to LDS; X's groups are stored chunk-fastest, so that a wave's
// chunks read contiguous bytes.  Products and sums are fp32 (v_dot2_f32_f16, as in
// the table path) in a fixed order.
//
// Bound by the random 16-byte codeword reads from LDS (about 80 bytes a clock
// per CU: 3.1 us for 17280 -> 960 with M = 4) and the launch and load latency
// before them.  One token, 17280 -> 960, M = 4: 7.5 us (table path 11.8); 512 ->
// 960, M = 2: 3.3 us (matrix cores 4.5).
#include <algorithm>

#include "aq_device.h"

namespace aq {

namespace {

constexpr int kFewWaves = 8;
constexpr int kFewAhead = 4;                   // rounds of codes loaded ahead
constexpr size_t kFewLdsBytes = 160 * 1024;

__device__ __forceinline__ half2v as_half2(uint32_t w) { return __builtin_bit_cast(half2v, w); }

// 8 fp16 values from 8 int8 values, exactly (1024 + (x + 128) minus 1152).
__device__ __forceinline__ u32x4 widen_i8(uint32_t lo, uint32_t hi) {
    lo ^= 0x80808080u;
    hi ^= 0x80808080u;
    const uint32_t k64 = 0x64646464u, bias = 0xE480E480u;
    return u32x4{add_f16x2(__builtin_amdgcn_perm(k64, lo, 0x04010400u), bias),
                 add_f16x2(__builtin_amdgcn_perm(k64, lo, 0x04030402u), bias),
                 add_f16x2(__builtin_amdgcn_perm(k64, hi, 0x04010400u), bias),
                 add_f16x2(__builtin_amdgcn_perm(k64, hi, 0x04030402u), bias)};
}

template <int XT, int MC, int NT, int R>
__global__ void __launch_bounds__(64 * kFewWaves, 2)
few_fwd_kernel(Geom geo, const u32x4* __restrict__ cb, const u32x4* __restrict__ codes,
               const float* __restrict__ scales, const void* __restrict__ X, const float* __restrict__ x_scales,
               void* __restrict__ Y, int y_dtype, int tiles) {
    constexpr int JC = 16 / MC;                  // groups per chunk
    constexpr int CL = 64 / R;                   // a wave's chunks
    constexpr int STEP = CL * kFewWaves;         // a workgroup's
    extern __shared__ __attribute__((aligned(16))) u32x4 lds_few[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntok = (int)geo.tokens;
    const int G = geo.G, nk = 1 << geo.B;
    const int nchunk = (G + JC - 1) / JC;
    // row tiles next to each other share code lines: keep them on one XCD
    const int per_xcd = (tiles + 7) / 8;
    const int tile = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
    if (tile >= tiles) return;

    const int row = tile * R + lane % R;
    const int rowc = min(row, geo.C_out - 1);    // rows past the last repeat it and are not stored
    const int c0 = CL * wave + lane / R;
    const __amdgpu_buffer_rsrc_t cr = buffer_rsrc(codes, (uint64_t)nchunk * geo.C_out * 16u);
    auto code_load = [&](int c) {                // (chunks past the last read zeros and are skipped)
        return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                             cr, c < nchunk ? ((uint32_t)c * (uint32_t)geo.C_out + (uint32_t)rowc) * 16u
                                                            : kOutOfRange, 0, 0));
    };
    u32x4 cw[kFewAhead];
#pragma unroll
    for (int i = 0; i < kFewAhead; ++i) cw[i] = code_load(c0 + STEP * i);

    // LDS: [MC][nk] codewords, one zero row, then x [NT][JC][nchunk] groups
    u32x4* cbl = lds_few;
    const int zero_row = MC * nk;
    u32x4* xl = lds_few + MC * nk + 1;
    for (int i = tid; i < MC * nk; i += 64 * kFewWaves) cbl[i] = cb[i];
    if (tid == 0) cbl[zero_row] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int n = 0; n < NT; ++n)
        for (int j = tid; j < nchunk * JC; j += 64 * kFewWaves) {
            u32x4 v{0u, 0u, 0u, 0u};
            if (n < ntok && j < G) {
                if constexpr (XT == AQ_I8) {
                    const uint32_t* p = reinterpret_cast<const uint32_t*>(static_cast<const int8_t*>(X) +
                                                                          ((int64_t)n * G + j) * 8);
                    v = widen_i8(p[0], p[1]);
                } else {
                    v = static_cast<const u32x4*>(X)[(int64_t)n * G + j];
                }
            }
            xl[((n * JC) + j % JC) * nchunk + j / JC] = v;
        }
    __syncthreads();

    float acc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[n] = 0.0f;
    for (int c = c0, r = 0; c < nchunk; c += STEP, ++r) {
        const u32x4 cur = cw[0];
#pragma unroll
        for (int i = 0; i + 1 < kFewAhead; ++i) cw[i] = cw[i + 1];
        cw[kFewAhead - 1] = code_load(c + STEP * kFewAhead);
#pragma unroll
        for (int jj = 0; jj < JC; ++jj) {
            u32x4 w[MC], xv[NT];
            const bool in = c * JC + jj < G;     // groups past K read the zero row
#pragma unroll
            for (int m = 0; m < MC; ++m) {
                const int i = jj * MC + m;
                const int code = (int)((cur[i >> 2] >> (8 * (i & 3))) & 0xFFu);
                w[m] = cbl[in ? m * nk + code : zero_row];
            }
#pragma unroll
            for (int n = 0; n < NT; ++n) xv[n] = xl[(n * JC + jj) * nchunk + c];
#pragma unroll
            for (int m = 0; m < MC; ++m)
#pragma unroll
                for (int d = 0; d < 4; ++d)
#pragma unroll
                    for (int n = 0; n < NT; ++n)
                        acc[n] = __builtin_amdgcn_fdot2(as_half2(xv[n][d]), as_half2(w[m][d]), acc[n], false);
        }
    }

    // the lanes of a row, then the waves in order
    __syncthreads();                             // X and the codebooks are done with
    float* red = reinterpret_cast<float*>(lds_few);
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        float v = acc[n];
#pragma unroll
        for (int o = R; o < 64; o *= 2) v += __shfl_xor(v, o, 64);
        if (lane < R) red[(wave * NT + n) * R + lane] = v;
    }
    __syncthreads();
    if (tid < R * NT) {
        const int n = tid / R, i = tile * R + tid % R;
        if (n < ntok && i < geo.C_out) {
            float v = red[tid];
#pragma unroll
            for (int w = 1; w < kFewWaves; ++w) v += red[w * NT * R + tid];
            v *= scales[i];
            if (x_scales) v *= x_scales[n];
            if (y_dtype == AQ_F32) store_y<AQ_F32>(Y, (int64_t)n * geo.C_out + i, v);
            else store_y<AQ_F16>(Y, (int64_t)n * geo.C_out + i, v);
        }
    }
}

size_t few_lds_bytes(const Geom& geo, int nt) {
    const int jc = 16 / geo.M;
    return (((size_t)geo.M << geo.B) + 1 + (size_t)nt * ((geo.G + jc - 1) / jc) * jc) * 16;
}

int few_nt(int64_t tokens) { return tokens == 1 ? 1 : tokens == 2 ? 2 : 4; }

template <int XT, int MC, int NT, int R>
hipError_t few_cfg(const Geom& geo, const DeviceWeights& w, const void* X, const float* xs, void* Y, int y_dtype,
                   hipStream_t st) {
    auto kern = few_fwd_kernel<XT, MC, NT, R>;
    const size_t lds = std::max<size_t>(few_lds_bytes(geo, NT), (size_t)kFewWaves * NT * R * sizeof(float));
    const hipError_t e = ensure_dynamic_lds((const void*)kern, lds);
    if (e != hipSuccess) return e;
    const int tiles = (geo.C_out + R - 1) / R;
    kern<<<8 * ((tiles + 7) / 8), 64 * kFewWaves, lds, st>>>(geo, static_cast<const u32x4*>(w.codebooks),
                                                             reinterpret_cast<const u32x4*>(w.codes_lut), w.scales, X, xs,
                                                             Y, y_dtype, tiles);
    note_launch(st, "few_fwd_kernel", {XT, MC, NT, R});
    return hipGetLastError();
}

// Rows per workgroup: the most that leave about three quarters of the compute
// units a workgroup each, and more where fewer rows give more workgroups than
// LDS holds at once (a last round of a few workgroups: 4 tokens, 13152 -> 1403,
// M = 1 14.7 us with 4 rows, 10.1 with 8; 17280 -> 2600 21.3 with 8, 15.6 with 16).
template <int XT, int MC, int NT>
hipError_t few_rows(const Geom& geo, const DeviceWeights& w, const void* X, const float* xs, void* Y, int y_dtype,
                    hipStream_t st) {
    const int64_t at_once = 256 * (int64_t)std::min<size_t>(2, kFewLdsBytes / few_lds_bytes(geo, NT));
    if (geo.C_out >= 16 * 192 || geo.C_out > 8 * at_once) return few_cfg<XT, MC, NT, 16>(geo, w, X, xs, Y, y_dtype, st);
    if (geo.C_out >= 8 * 192 || geo.C_out > 4 * at_once) return few_cfg<XT, MC, NT, 8>(geo, w, X, xs, Y, y_dtype, st);
    return few_cfg<XT, MC, NT, 4>(geo, w, X, xs, Y, y_dtype, st);
}

template <int XT, int MC>
hipError_t few_tokens(const Geom& geo, const DeviceWeights& w, const void* X, const float* xs, void* Y, int y_dtype,
                      hipStream_t st) {
    switch (few_nt(geo.tokens)) {
    case 1: return few_rows<XT, MC, 1>(geo, w, X, xs, Y, y_dtype, st);
    case 2: return few_rows<XT, MC, 2>(geo, w, X, xs, Y, y_dtype, st);
    default: return few_rows<XT, MC, 4>(geo, w, X, xs, Y, y_dtype, st);
    }
}

template <int XT>
hipError_t few_books(const Geom& geo, const DeviceWeights& w, const void* X, const float* xs, void* Y, int y_dtype,
                     hipStream_t st) {
    switch (geo.M) {
    case 1: return few_tokens<XT, 1>(geo, w, X, xs, Y, y_dtype, st);
    case 2: return few_tokens<XT, 2>(geo, w, X, xs, Y, y_dtype, st);
    case 4: return few_tokens<XT, 4>(geo, w, X, xs, Y, y_dtype, st);
    default: return hipErrorInvalidConfiguration;
    }
}

}  // namespace

bool few_supported(const Geom& geo, int cb_dtype, int x_dtype) {
    if (geo.conv || geo.g != 8 || geo.B > 8 || cb_dtype != AQ_F16) return false;
    if (geo.M != 1 && geo.M != 2 && geo.M != 4) return false;
    if (x_dtype != AQ_F16 && x_dtype != AQ_I8) return false;
    if (geo.tokens > 4 || few_lds_bytes(geo, few_nt(geo.tokens)) > kFewLdsBytes) return false;
    return (int64_t)(geo.G * (int64_t)geo.M / 16 + 1) * geo.C_out * 16 < (int64_t(1) << 31);   // 32-bit code offsets
}

hipError_t launch_few_forward(const Geom& geo, const DeviceWeights& w, const void* X, int x_dtype,
                              const float* x_scales, void* Y, int y_dtype, hipStream_t stream) {
    if (x_dtype == AQ_I8) return few_books<AQ_I8>(geo, w, X, x_scales, Y, y_dtype, stream);
    return few_books<AQ_F16>(geo, w, X, x_scales, Y, y_dtype, stream);
}

}  // namespace aq
