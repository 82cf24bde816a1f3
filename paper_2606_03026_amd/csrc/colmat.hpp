// Matrix-core contraction read straight from the column-major weights, for
// many spike rows against one weight matrix without a packed copy of it
// (gfx950 v_mfma_i32_16x16x64_i8).
//
// The stream's tokens that use the same weight copy are the rows of one
// batch: acc[t][n] = sum_k x[t][k] Q[n][k] with x in {0,1}.  The gather reads
// every active column once per token; here a weight byte is read once per
// 64 tokens.  Products are 0 or a weight and INT32 sums are exact, so the
// results have the gather's bits.
//
// Operands.  A step is 64 of the 128 columns of a double step; lane
// 16 q + c holds, of 8 consecutive channels 8 c .. 8 c + 7 of the wave's 128,
// the 16 columns 32 q + i + 8 m (m = 0..3; i = 0..3 in a double step's first
// step, 4..7 in its second): 16 loads of 8 bytes, each instruction reading 128
// contiguous bytes of four columns.  4 x 4 byte transposes (v_perm_b32) turn
// them into the operands of the 8 channels: byte m of dword i holds column
// 32 q + i + 8 m.  With that column order one dword of the mask (bits
// 32 q .. 32 q + 31 of the double step) gives the spike operand of a row by a
// shift and an AND per dword: (bits >> i) & 0x01010101.  Bits past K meet
// columns past the end of W, which read as zero.
//
// Work split.  A workgroup of 4 waves owns up to 64 tokens of one weight
// matrix and 128 channels; its waves take every fourth double step, keep two
// steps (16 KB) of weights in flight each, and add their sums through LDS,
// each wave finishing a quarter of the token rows.  Tiles go longest K first,
// dealt to the XCDs in turn (one tile at a time: a whole projection at a time
// left some XCDs 9% more work; where rows are not whole 128-byte lines, a
// projection's tiles stay on one XCD, whose L2 serves the lines they share).
// The token tiles of one weight tile run side by side on one XCD.
//
// It is bound by HBM: 250 tokens over 4 copies of 44 projections (1.04 GB of
// weights, 68 MB of results) take 212 us, 5.2 TB/s (the gather 1346 us); 30 us
// of that are the stores (182 us with them switched off in a timing copy), and
// a plain nontemporal read of 1 GiB takes 155 us.  Spike dwords read from
// global memory with each double step instead of staged in LDS, and sums
// stored 16 bytes of every 32 at a time, took 241 us; the matrix and vector
// units are busy about 26 and 20 us of it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "buffer.hpp"
#include "gather.hpp"

namespace spk {

constexpr int kColWaves = 4;
constexpr int kColBlock = 64 * kColWaves;
constexpr int kColChannels = 128;  // channels of a workgroup
constexpr int kColStep = 128;      // columns of a double step (two mask words)

// Rows of four channels' bytes -> per channel the four rows' bytes.
__device__ inline void transpose_bytes(const uint32_t (&r)[4], uint32_t (&ch)[4])
{
    const uint32_t lo01 = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u), hi01 = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);
    const uint32_t lo23 = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u), hi23 = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
    ch[0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
    ch[1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
    ch[2] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
    ch[3] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
}

// The stream's projections for the matrix cores: items are (weight set, projection) pairs,
// item i = set i % n_sets of projection order[i / n_sets] (longest K first).
struct ColumnOrder {
    uint8_t proj[kStreamMaxProj];
};

// LDS of a workgroup: its rows' spike words, later its waves' sums.  Rows of
// staged words are an odd number of 16-byte units apart (rounded up to whole
// double steps), so the 16 rows that one operand read touches lie in distinct
// banks.
__host__ __device__ constexpr int column_row_units(int K) { return (K + kColStep - 1) / kColStep | 1; }
constexpr int column_round(int RT) { return RT < 2 ? RT : 2; }  // (row subtile, register) pairs of a wave's share in LDS at once
inline int column_lds(int RT, int K)
{
    const int words = 16 * RT * column_row_units(K) * 16;
    const int sums = kColWaves * kColWaves * column_round(RT) * 2048;
    return words > sums ? words : sums;
}

// 16 RT tokens x 128 channels of one item per workgroup.  NT: weight loads
// marked nontemporal.
template <int RT, bool NT>
__global__ __launch_bounds__(kColBlock) __attribute__((amdgpu_waves_per_eu(RT == 1 ? 4 : RT == 2 ? 3 : 2))) void k_stream_mat(
    const StreamOperands* __restrict__ desc, const StreamLayout layout, const ColumnOrder order, int n_proj,
    int n_sets, int n_tokens, int N, int n_coltiles, int n_rowtiles, const uint64_t* __restrict__ masks,
    int mask_stride, float* __restrict__ out, int64_t out_stride)
{
    typedef int32_t acc_t __attribute__((ext_vector_type(4)));
    constexpr int kPairs = RT;  // (row subtile, register) pairs a wave finishes
    constexpr int kRound = column_round(RT);
    extern __shared__ __align__(16) uint8_t lds[];

    // Workgroup b runs on XCD b % 8.
    const int used_sets = min(n_sets, n_tokens);
    const int b = blockIdx.x / 8, xcd = blockIdx.x % 8;
    int item, ct;
    if (N % kColChannels == 0) {
        const int pair = b / n_rowtiles * 8 + xcd;
        item = pair / n_coltiles;
        ct = pair % n_coltiles;
    } else {
        const int tile = b / n_rowtiles;
        item = tile / n_coltiles * 8 + xcd;
        ct = tile % n_coltiles;
    }
    if (item >= used_sets * n_proj)
        return;
    const int n0 = ct * kColChannels;
    const int row0 = b % n_rowtiles * 16 * RT;
    const int set = item % used_sets;
    const int proj = order.proj[item / used_sets];
    const int K = layout.K[proj];
    const StreamOperands ops = desc[set * n_proj + proj];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int l = threadIdx.x % 64;
    const int q = l / 16;  // column group of the operands, row group of the result
    const int c = l % 16;  // token row of the spikes, 8-channel group of the weights and the result
    const __amdgpu_buffer_rsrc_t wres = weight_resource(ops.W, (int64_t)K * N);
    const int w_bytes = K * N;
    const int n_double = (K + kColStep - 1) / kColStep;

    // A column past the end of W (also of a double step past the wave's last)
    // is read at the end of the resource: zeros, without a memory request.  (A
    // scalar offset beyond that end would wrap the hardware's range check.)
    const uint32_t w_off = (uint32_t)(32 * q * N + n0 + 8 * c);
    auto load_weights = [&](int d, int half, u32x2 (&w)[16]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int k = kColStep * d + 4 * half + i + 8 * m;
                w[4 * i + m] = __builtin_amdgcn_raw_buffer_load_b64(wres, w_off, k < K ? k * N : w_bytes, NT ? 2 : 0);
            }
    };
    u32x2 w0[16], w1[16];
    load_weights(wave, 0, w0);
    load_weights(wave, 1, w1);

    // The rows' spike words, whole double steps of them: the last one's upper
    // word may be the next row's, whose bits meet zero weights.
    const int units = column_row_units(K);
    {
        const __amdgpu_buffer_rsrc_t mres = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint64_t*>(masks), 0, n_tokens * mask_stride * (int)sizeof(uint64_t), kBufferFlags);
        uint64_t* words = reinterpret_cast<uint64_t*>(lds);
        const int total = 16 * RT * 2 * n_double;
        constexpr int kBatch = 8;
        for (int base = threadIdx.x; base < total; base += kBatch * kColBlock) {
            u32x2 v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int e = base + u * kColBlock;
                const int r = e / (2 * n_double), w = e - r * 2 * n_double;
                const int64_t t = (int64_t)(row0 + r) * n_sets + set;
                const uint32_t off =
                    e < total && t < n_tokens ? (uint32_t)(t * mask_stride + layout.mask_off[proj] + w) * 8u : kOutOfRange;
                v[u] = __builtin_amdgcn_raw_buffer_load_b64(mres, off, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int e = base + u * kColBlock;
                const int r = e / (2 * n_double), w = e - r * 2 * n_double;
                if (e < total)
                    words[r * 2 * units + w] = __builtin_bit_cast(uint64_t, v[u]);
            }
        }
        __syncthreads();
    }
    auto read_bits = [&](int d, uint32_t (&bits)[RT]) {
        const uint32_t* dwords = reinterpret_cast<const uint32_t*>(lds);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
            bits[rt] = dwords[((16 * rt + c) * units + d) * 4 + q];
    };

    acc_t acc[RT][8];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < 8; ++t)
            acc[rt][t] = acc_t{0, 0, 0, 0};
    auto products = [&](const uint32_t (&bits)[RT], int half, const u32x2 (&w)[16]) {
        acc_t a[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                a[rt][i] = (int32_t)((bits[rt] >> (4 * half + i)) & 0x01010101u);
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // channels 8 c + 4 h .. 8 c + 4 h + 3
            uint32_t ch[4][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t r[4] = {w[4 * i][h], w[4 * i + 1][h], w[4 * i + 2][h], w[4 * i + 3][h]};
                transpose_bytes(r, ch[i]);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const acc_t bw = {(int32_t)ch[0][t], (int32_t)ch[1][t], (int32_t)ch[2][t], (int32_t)ch[3][t]};
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    acc[rt][4 * h + t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[rt], bw, acc[rt][4 * h + t], 0, 0, 0);
            }
        }
    };

    for (int d = wave; d < n_double; d += kColWaves) {
        uint32_t bits[RT];
        read_bits(d, bits);
        products(bits, 0, w0);
        load_weights(d + kColWaves, 0, w0);
        __builtin_amdgcn_sched_barrier(0);
        products(bits, 1, w1);
        load_weights(d + kColWaves, 1, w1);
        __builtin_amdgcn_sched_barrier(0);
    }

    // Register j of lane 16 q + c of acc[rt][t]: token row 16 rt + 4 q + j,
    // channel 8 c + t.  Pair p = 4 rt + j (four rows) belongs to wave
    // p / kPairs, which adds the four waves' sums from LDS, kRound pairs at a
    // time.  A lane's two 16-byte halves (channels 8 c + 4 h ..) lie side by
    // side, swapped in every second group of four lanes (no two lanes of a
    // write share a bank); read back in channel order, every store instruction
    // writes whole runs of 512 bytes of two rows.
    i32x4* part = reinterpret_cast<i32x4*>(lds);  // [owner][source][kRound][64 lanes][2]
    auto half_at = [](int owner, int source, int i, int lane, int h) {
        return (((owner * kColWaves + source) * kRound + i) * 64 + lane) * 2 + (h ^ ((lane >> 2) & 1));
    };
#pragma unroll
    for (int p0 = 0; p0 < kPairs; p0 += kRound) {
        __syncthreads();  // spike words or the pairs before have been read
#pragma unroll
        for (int w = 0; w < kColWaves; ++w)
#pragma unroll
            for (int i = 0; i < kRound; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int p = w * kPairs + p0 + i, rt = p / 4, j = p % 4;
                    part[half_at(w, wave, i, l, h)] =
                        i32x4{acc[rt][4 * h][j], acc[rt][4 * h + 1][j], acc[rt][4 * h + 2][j], acc[rt][4 * h + 3][j]};
                }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kRound; ++i)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int p = wave * kPairs + p0 + i, rt = p / 4, j = p % 4;
                const int qr = l / 32 + 2 * g, c4 = l % 32;  // row group, group of four channels
                const int64_t t = (int64_t)(row0 + 16 * rt + 4 * qr + j) * n_sets + set;
                const int n = n0 + 4 * c4;
                if (t >= n_tokens || n >= N)
                    continue;
                i32x4 sum = part[half_at(wave, 0, i, 16 * qr + c4 / 2, c4 % 2)];
#pragma unroll
                for (int s = 1; s < kColWaves; ++s)
                    sum += part[half_at(wave, s, i, 16 * qr + c4 / 2, c4 % 2)];
                float* o = out + t * out_stride + (int64_t)proj * N + n;
                const float* sc = ops.scale + n;
                f32x4 y;  // per channel: one conversion (exact below 2^24, RNE beyond), one binary32 multiply
                if (((reinterpret_cast<uintptr_t>(o) | reinterpret_cast<uintptr_t>(sc)) & 15) == 0) {
                    const f32x4 s4 = *reinterpret_cast<const f32x4*>(sc);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        y[e] = (float)sum[e] * s4[e];
                    __builtin_nontemporal_store(y, reinterpret_cast<f32x4*>(o));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        o[e] = (float)sum[e] * sc[e];
                }
            }
    }
}

}  // namespace spk
