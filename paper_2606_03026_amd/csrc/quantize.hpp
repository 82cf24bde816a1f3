// Symmetric per-output-channel INT8 quantization and export (gfx950).
//
// For a weight matrix W [M][K] (row m = output channel m), paper Sec. 2.3:
//
//     s_m     = max(max_k |W[m][k]|, 1e-8) / 127
//     Q[m][k] = clip(round(W[m][k] / s_m), -127, 127)
//
// in binary32: the maximum is exact, both divisions are correctly rounded
// (v_div_scale / v_div_fmas / v_div_fixup; quantize_four leaves one out only
// where it is shown to decide nothing), and round() is v_rndne (ties to even).  Q is written row-major (the dense
// continuous-input layout) or column-major (W_cm[k][m] = Q[m][k], the
// spike-gated layout, Sec. 2.2).
//
// Rows of at most 4096 values (K % 4 == 0, aligned) take one pass:
// k_quant_rows for the row-major layout -- one wave per row holds the row in
// registers, reduces its maximum over the wave, writes s and the row of Q --
// and k_quant_cols for the column-major one where there are rows enough.
// Otherwise two passes, both bound by HBM: k_quant_scale (one wave per row) or
// k_quant_scale_row (one workgroup per row) reads each row once and writes s;
// k_quant_tile reads W again in 64 x 64 tiles, quantizes, and writes Q.  For
// the column-major layout the tile is transposed through LDS so that both the
// reads (along k) and the writes (along m) are contiguous.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bytes.hpp"

namespace spk {

constexpr int kQuantBlock = 256;
constexpr int kQuantTile = 64;  // rows (m) and columns (k) of a tile

// one wave per row: s[m] from the row's largest magnitude.  VEC (K % 4 == 0,
// W 16-byte aligned): 16-byte loads; either way 8 loads per lane are in
// flight before any is used.
template <bool VEC>
__global__ __launch_bounds__(kQuantBlock) void k_quant_scale(const float* __restrict__ W, int M, int K,
                                                             float* __restrict__ scale)
{
    const int lane = threadIdx.x % 64;
    const int m = blockIdx.x * (kQuantBlock / 64) + threadIdx.x / 64;
    if (m >= M)
        return;
    const float* row = W + (int64_t)m * K;
    constexpr int kBatch = 8;
    float amax = 0.0f;
    if constexpr (VEC) {
        const float4* row4 = reinterpret_cast<const float4*>(row);
        const int n4 = K / 4;
        for (int c0 = lane; c0 < n4; c0 += 64 * kBatch) {
            float4 v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int c = c0 + 64 * u;
                v[u] = c < n4 ? row4[c] : float4{0.0f, 0.0f, 0.0f, 0.0f};
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v[u].x), fabsf(v[u].y)), fmaxf(fabsf(v[u].z), fabsf(v[u].w))));
        }
    } else {
        for (int k0 = lane; k0 < K; k0 += 64 * kBatch) {
            float v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int k = k0 + 64 * u;
                v[u] = k < K ? row[k] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                amax = fmaxf(amax, fabsf(v[u]));
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
        amax = fmaxf(amax, __shfl_xor(amax, d, 64));
    if (lane == 0)
        scale[m] = __fdiv_rn(fmaxf(amax, 1e-8f), 127.0f);
}

// The same with a whole workgroup per row (K % 4 == 0, W 16-byte aligned): one
// wave per row walks a long row in turns and leaves the chip short of loads in
// flight (1536 x 6144: 10.8 us; here 7.9, 4.8 TB/s).
__global__ __launch_bounds__(kQuantBlock) void k_quant_scale_row(const float* __restrict__ W, int K,
                                                                 float* __restrict__ scale)
{
    __shared__ float wave_max[kQuantBlock / 64];
    const float4* row4 = reinterpret_cast<const float4*>(W + (int64_t)blockIdx.x * K);
    constexpr int kBatch = 8;
    const int n4 = K / 4;
    float amax = 0.0f;
    for (int c0 = threadIdx.x; c0 < n4; c0 += kQuantBlock * kBatch) {
        float4 v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int c = c0 + kQuantBlock * u;
            v[u] = c < n4 ? row4[c] : float4{0.0f, 0.0f, 0.0f, 0.0f};
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v[u].x), fabsf(v[u].y)), fmaxf(fabsf(v[u].z), fabsf(v[u].w))));
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
        amax = fmaxf(amax, __shfl_xor(amax, d, 64));
    if (threadIdx.x % 64 == 0)
        wave_max[threadIdx.x / 64] = amax;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kQuantBlock / 64; ++w)
            amax = fmaxf(amax, wave_max[w]);
        scale[blockIdx.x] = __fdiv_rn(fmaxf(amax, 1e-8f), 127.0f);
    }
}

__device__ inline int8_t quantize_one(float w, float s)
{
    const float r = __builtin_rintf(__fdiv_rn(w, s));
    return (int8_t)fminf(fmaxf(r, -127.0f), 127.0f);
}

// Codes of four weights of one row as four bytes, rn = fl32(1 / s).
//
// The correctly rounded division costs about ten instructions, more than the
// rest of the export, and decides nothing unless w / s lies next to a tie:
// u = fma(w, rn, 1.5 * 2^23) has the integer nearest to w rn in its low bits
// (as two's complement), and e = w rn - n is what is left.  With |w / s| <=
// 127 (1 + 2^-23), w rn differs from w / s by at most 127 * 2^-24 * (1 + 2^-22)
// and fl32(w / s) by at most 2^-18, together below 2^-16; so where |e| <= 1/2 - 2^-15,
// rint(fl32(w / s)) is n.  Elsewhere (one weight in 16,000; also NaN, and rows
// whose scale is not finite) the definition itself is evaluated.  s is at
// least 1e-8 / 127, so rn is finite and normal wherever s is.
__device__ inline uint32_t quantize_four(const float4& w, float s, float rn)
{
    constexpr float kMagic = 12582912.0f, kSure = 0.5f - 0x1p-15f;
    const float v[4] = {w.x, w.y, w.z, w.w};
    uint32_t u[4];
    bool sure = true;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float m = __builtin_fmaf(v[i], rn, kMagic);
        const float e = __builtin_fmaf(v[i], rn, kMagic - m);
        sure = sure && fabsf(e) <= kSure;
        u[i] = __builtin_bit_cast(uint32_t, m);
    }
    if (!sure) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            u[i] = (uint32_t)(int32_t)quantize_one(v[i], s);
    }
    const uint32_t lo = __builtin_amdgcn_perm(u[1], u[0], 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm(u[3], u[2], 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// One wave per row, the row in registers: lane l holds the float4 chunks
// l + 64 j (j < NV) of its row, so K <= 256 NV.  Needs K % 4 == 0, W 16-byte
// and Q 4-byte aligned (host-checked).
constexpr int kQuantRowsMaxK = 4096;
template <int NV>
__global__ __launch_bounds__(kQuantBlock) void k_quant_rows(const float* __restrict__ W, int M, int K,
                                                            int8_t* __restrict__ Q, float* __restrict__ scale)
{
    const int lane = threadIdx.x % 64;
    const int m = blockIdx.x * (kQuantBlock / 64) + threadIdx.x / 64;
    if (m >= M)
        return;
    const int n4 = K / 4;
    const float4* row = reinterpret_cast<const float4*>(W + (int64_t)m * K);
    float4 w[NV];
    float amax = 0.0f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = lane + 64 * j;
        w[j] = c < n4 ? row[c] : float4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int j = 0; j < NV; ++j)
        amax = fmaxf(amax, fmaxf(fmaxf(fabsf(w[j].x), fabsf(w[j].y)), fmaxf(fabsf(w[j].z), fabsf(w[j].w))));
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
        amax = fmaxf(amax, __shfl_xor(amax, d, 64));
    const float s = __fdiv_rn(fmaxf(amax, 1e-8f), 127.0f);
    if (lane == 0)
        scale[m] = s;
    const float rn = __fdiv_rn(1.0f, s);
    uint32_t* dst = reinterpret_cast<uint32_t*>(Q + (int64_t)m * K);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = lane + 64 * j;
        if (c < n4)
            dst[c] = quantize_four(w[j], s, rn);
    }
}

// Column-major export in one pass: a workgroup of 16 waves takes 16
// consecutive rows, one per wave and held in its registers (lane l: float4
// chunks l + 64 j, j < NV, so K <= 256 NV), reduces each row's maximum, writes
// s, and leaves the codes in LDS as 16 rows of K bytes; then each thread takes
// four columns, transposes their 16 x 4 codes in registers and writes 16
// consecutive bytes of each column.  Consecutive row groups run on one XCD,
// whose L2 merges their pieces of a column into whole lines.  Needs K % 4 ==
// 0, M % 16 == 0, W and Q 16-byte aligned (host-checked), 16 K bytes of
// dynamic LDS.
//
// Bound by HBM while every CU has rows of its own: 8192 x 1152 takes 11.1 us
// (4.2 TB/s; two passes 17.4), 6144 x 1536 11.8 (17.0).  With 8 rows the
// pieces of 8 bytes cost more in stores than the shorter reads give back
// (13.4 us for both).
constexpr int kColRows = 16;
template <int NV>
__global__ __launch_bounds__(64 * kColRows) void k_quant_cols(const float* __restrict__ W, int M, int K,
                                                       int8_t* __restrict__ Q, float* __restrict__ scale)
{
    extern __shared__ __align__(16) uint32_t codes[];  // [16][K / 4]
    const int lane = threadIdx.x % 64, r = threadIdx.x / 64;
    const int groups = M / kColRows, per = (groups + 7) / 8;
    const int g = (int)(blockIdx.x % 8) * per + blockIdx.x / 8;
    if ((int)(blockIdx.x / 8) >= per || g >= groups)  // the whole workgroup
        return;
    const int m = g * kColRows + r;
    const int n4 = K / 4;
    const float4* row = reinterpret_cast<const float4*>(W + (int64_t)m * K);
    float4 w[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = lane + 64 * j;
        w[j] = c < n4 ? row[c] : float4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    float amax = 0.0f;
#pragma unroll
    for (int j = 0; j < NV; ++j)
        amax = fmaxf(amax, fmaxf(fmaxf(fabsf(w[j].x), fabsf(w[j].y)), fmaxf(fabsf(w[j].z), fabsf(w[j].w))));
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
        amax = fmaxf(amax, __shfl_xor(amax, d, 64));
    const float s = __fdiv_rn(fmaxf(amax, 1e-8f), 127.0f);
    if (lane == 0)
        scale[m] = s;
    const float rn = __fdiv_rn(1.0f, s);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = lane + 64 * j;
        if (c < n4)
            codes[r * n4 + c] = quantize_four(w[j], s, rn);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < n4; c += 64 * kColRows) {
        uint32_t out[4][kColRows / 4];  // [column of the four][rows 4 i .. 4 i + 3]
#pragma unroll
        for (int i = 0; i < kColRows / 4; ++i) {
            uint32_t d[4], t[4];
#pragma unroll
            for (int a = 0; a < 4; ++a)
                d[a] = codes[(4 * i + a) * n4 + c];
            transpose_bytes(d, t);
#pragma unroll
            for (int a = 0; a < 4; ++a)
                out[a][i] = t[a];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            int8_t* dst = Q + (int64_t)(4 * c + k) * M + g * kColRows;
            *reinterpret_cast<uint4*>(dst) = uint4{out[k][0], out[k][1], out[k][2], out[k][3]};
        }
    }
}

// One 64 x 64 tile (rows m0.., columns k0..) per workgroup.  Each thread
// takes 4 consecutive columns of 4 rows.  COL: write W_cm[k][m] through an
// LDS transpose, 4 consecutive m per thread.  VEC (host-checked: K % 4 == 0,
// W 16-byte aligned, Q 4-byte aligned, and M % 4 == 0 for COL): 16-byte
// loads of W and 4-byte stores of Q; otherwise element by element.
template <bool COL, bool VEC>
__global__ __launch_bounds__(kQuantBlock) void k_quant_tile(const float* __restrict__ W, const float* __restrict__ scale,
                                                            int M, int K, int8_t* __restrict__ Q, int tiles_k)
{
    __shared__ __align__(16) int8_t tile[kQuantTile][kQuantTile + 4];  // [k][m] for COL
    const int m0 = (blockIdx.x / tiles_k) * kQuantTile;
    const int k0 = (blockIdx.x % tiles_k) * kQuantTile;
    const int c4 = (threadIdx.x % 16) * 4;  // first of the thread's 4 columns
    const int r0 = threadIdx.x / 16;        // rows r0 + 16 i
#pragma unroll
    for (int i = 0; i < kQuantTile / 16; ++i) {
        const int r = r0 + 16 * i;
        const int m = m0 + r, k = k0 + c4;
        int8_t q[4] = {0, 0, 0, 0};
        if (m < M) {
            const float s = scale[m];
            const float* src = W + (int64_t)m * K + k;
            if (VEC && k + 3 < K) {
                const uint32_t d = quantize_four(*reinterpret_cast<const float4*>(src), s, __fdiv_rn(1.0f, s));
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    q[j] = (int8_t)(d >> (8 * j));
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (k + j < K)
                        q[j] = quantize_one(src[j], s);
            }
        }
        if constexpr (COL) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                tile[c4 + j][r] = q[j];
        } else if (m < M) {
            int8_t* dst = Q + (int64_t)m * K + k;
            if (VEC && k + 3 < K) {
                *reinterpret_cast<uint32_t*>(dst) = (uint32_t)(uint8_t)q[0] | (uint32_t)(uint8_t)q[1] << 8 |
                                                    (uint32_t)(uint8_t)q[2] << 16 | (uint32_t)(uint8_t)q[3] << 24;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (k + j < K)
                        dst[j] = q[j];
            }
        }
    }
    if constexpr (COL) {
        __syncthreads();
        // thread: 4 consecutive m (mm .. mm + 3) of the tile's columns kk
#pragma unroll
        for (int i = 0; i < kQuantTile / 16; ++i) {
            const int kk = r0 + 16 * i;
            const int k = k0 + kk, m = m0 + c4;
            if (k >= K)
                continue;
            int8_t* dst = Q + (int64_t)k * M + m;
            if (VEC && m + 3 < M) {
                *reinterpret_cast<uint32_t*>(dst) = *reinterpret_cast<const uint32_t*>(&tile[kk][c4]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (m + j < M)
                        dst[j] = tile[kk][c4 + j];
            }
        }
    }
}

}  // namespace spk
