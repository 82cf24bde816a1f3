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

#include <algorithm>

#include "buffer.hpp"
#include "gather.hpp"
#include "mfma.hpp"  // mf_i32x4

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

// Four channels' outputs: per channel one conversion (exact below 2^24, RNE
// beyond) and one binary32 multiply.
__device__ inline void store_channels(i32x4 sum, float* o, const float* __restrict__ sc)
{
    if (((reinterpret_cast<uintptr_t>(o) | reinterpret_cast<uintptr_t>(sc)) & 15) == 0) {
        const f32x4 s4 = *reinterpret_cast<const f32x4*>(sc);
        f32x4 y;
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

// The sums of a workgroup's waves, scaled and stored.  Register j of lane
// 16 q + c of acc[rt][t] is row 16 rt + 4 q + j, channel n0 + 8 c + t; row_of(r)
// gives row r's outputs (null: none).
//
// Pair p = 4 rt + j (four rows) belongs to wave p / RT, which adds the four
// waves' sums from LDS, column_round(RT) pairs at a time.  A lane's two 16-byte
// halves (channels 8 c + 4 h ..) lie side by side, swapped in every second
// group of four lanes (no two lanes of a write share a bank); read back in
// channel order, every store instruction writes whole runs of 512 bytes of
// two rows.
template <int RT, class RowOf>
__device__ inline void finish_column_tile(const mf_i32x4 (&acc)[RT][8], int wave, int l, int n0, int N,
                                          const float* __restrict__ scale, uint8_t* lds, RowOf row_of)
{
    constexpr int kPairs = RT;
    constexpr int kRound = column_round(RT);
    i32x4* part = reinterpret_cast<i32x4*>(lds);  // [owner][source][kRound][64 lanes][2]
    auto half_at = [](int owner, int source, int i, int lane, int h) {
        return (((owner * kColWaves + source) * kRound + i) * 64 + lane) * 2 + (h ^ ((lane >> 2) & 1));
    };
#pragma unroll
    for (int p0 = 0; p0 < kPairs; p0 += kRound) {
        __syncthreads();  // what lay in LDS has been read
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
                const int n = n0 + 4 * c4;
                float* o = row_of(16 * rt + 4 * qr + j);
                if (!o || n >= N)
                    continue;
                o += n;
                i32x4 sum = part[half_at(wave, 0, i, 16 * qr + c4 / 2, c4 % 2)];
#pragma unroll
                for (int s = 1; s < kColWaves; ++s)
                    sum += part[half_at(wave, s, i, 16 * qr + c4 / 2, c4 % 2)];
                store_channels(sum, o, scale + n);
            }
    }
}

// 16 RT tokens x 128 channels of one item per workgroup.  NT: weight loads
// marked nontemporal.
template <int RT, bool NT>
__global__ __launch_bounds__(kColBlock) __attribute__((amdgpu_waves_per_eu(RT == 1 ? 4 : RT == 2 ? 3 : 2))) void k_stream_mat(
    const StreamOperands* __restrict__ desc, const StreamLayout layout, const ColumnOrder order, int n_proj,
    int n_sets, int n_tokens, int N, int n_coltiles, int n_rowtiles, const uint64_t* __restrict__ masks,
    int mask_stride, float* __restrict__ out, int64_t out_stride)
{
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
    const uint32_t w_off = n0 + 8 * c < N ? (uint32_t)(32 * q * N + n0 + 8 * c) : kOutOfRange;  // channels past N: no request
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

    mf_i32x4 acc[RT][8];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < 8; ++t)
            acc[rt][t] = mf_i32x4{0, 0, 0, 0};
    auto products = [&](const uint32_t (&bits)[RT], int half, const u32x2 (&w)[16]) {
        mf_i32x4 a[RT];
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
                const mf_i32x4 bw = {(int32_t)ch[0][t], (int32_t)ch[1][t], (int32_t)ch[2][t], (int32_t)ch[3][t]};
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

    finish_column_tile<RT>(acc, wave, l, n0, N, ops.scale, lds, [&](int r) -> float* {
        const int64_t t = (int64_t)(row0 + r) * n_sets + set;
        return t < n_tokens ? out + t * out_stride + (int64_t)proj * N : nullptr;
    });
}

// ---------------------------------------------------------------------------
// The same contraction over the columns that are active in any of up to 8
// rows: at a rate of 0.1 seven rows touch half the columns, one row a tenth,
// and the others' weights are not read.
//
// The union of the rows' spikes becomes a list of columns in LDS with a byte
// per column holding which rows are active there (an 8 x 8 bit transpose of
// the rows' bytes).  A step is 64 entries of the list, lane 16 q + c taking
// entries 16 q .. 16 q + 15: its weight loads go to those columns, and the
// spike operand of row c is bit c of the entries' row bytes, a shift and an
// AND per four columns.  Entries past the list name column K, whose weights
// read as zero.  Everything else is as above, but with 8 waves to a workgroup.
//
// What bounds it is the random 128-byte reads: 7 rows of the 44-projection
// stack, 143 MB of active columns, take 38 us, of which 8 are the launch, the
// lists and the sums (a timing copy with one step per wave); 4 waves a
// workgroup take 40, and wider tiles (2 or 3 x 128 channels sharing a list)
// 44 and 50: half as many workgroups leave compute units idle.
// ---------------------------------------------------------------------------
constexpr int kActiveMaxRows = 8;
constexpr int kActiveMaxK = 64 * kMaxSliceWords;
constexpr int kActiveWaves = 8;
constexpr int kActiveBlock = 64 * kActiveWaves;
constexpr int kActiveStep = 64;
// list (16-bit columns) and row bytes, padded by the step read past the end;
// later the waves' sums of the 8 rows
inline int active_lds(int K)
{
    const int entries = (K + kActiveStep - 1) / kActiveStep * kActiveStep + kActiveStep;
    return std::max(3 * entries, kActiveWaves * kActiveMaxRows * kColChannels * (int)sizeof(int32_t));
}

// Byte b of x holds eight columns of row b; afterwards byte i holds the rows of column i.
__device__ inline uint64_t transpose_bits(uint64_t x)
{
    uint64_t t = (x ^ (x >> 7)) & 0x00AA00AA00AA00AAull;
    x ^= t ^ (t << 7);
    t = (x ^ (x >> 14)) & 0x0000CCCC0000CCCCull;
    x ^= t ^ (t << 14);
    t = (x ^ (x >> 28)) & 0x00000000F0F0F0F0ull;
    return x ^ t ^ (t << 28);
}

// One workgroup: n_rows rows (spike row r at byte mask0 + r * mask_pitch of
// the resource mres) against channels n0 .. n0 + 127 of W.
template <bool NT, class RowOf>
__device__ __attribute__((always_inline)) inline void active_tile(const int8_t* W, const float* scale, int K, int N, int n0,
                                                                  __amdgpu_buffer_rsrc_t mres, uint32_t mask0,
                                                                  uint32_t mask_pitch, int n_rows, uint8_t* lds,
                                                                  RowOf row_of)
{
    __shared__ int wave_total[kActiveWaves];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int l = threadIdx.x % 64;
    const int q = l / 16;  // entry group of the operands, row group of the result
    const int c = l % 16;  // row of the spikes, 8-channel group of the weights and the result
    const int entries = (K + kActiveStep - 1) / kActiveStep * kActiveStep + kActiveStep;
    uint16_t* list = reinterpret_cast<uint16_t*>(lds);
    uint8_t* rows = lds + 2 * entries;

    // Compaction, 16 columns per thread (8192 per pass).
    int cnt = 0;
    for (int k0 = 0; k0 < K; k0 += 16 * kActiveBlock) {
        const int kt = k0 + 16 * (int)threadIdx.x;  // this thread's first column
        uint32_t d[kActiveMaxRows];
#pragma unroll
        for (int r = 0; r < kActiveMaxRows; ++r)
            d[r] = __builtin_amdgcn_raw_buffer_load_b16(
                mres, r < n_rows && kt < K ? mask0 + r * mask_pitch + (uint32_t)kt / 8 : kOutOfRange, 0, 0);
        const uint32_t valid = K - kt >= 16 ? 0xffffu : kt < K ? (1u << (K - kt)) - 1u : 0u;
        uint64_t byte_rows[2] = {0, 0};
        uint32_t any = 0;
#pragma unroll
        for (int r = 0; r < kActiveMaxRows; ++r) {
            d[r] &= valid;
            any |= d[r];
            byte_rows[0] |= (uint64_t)(d[r] & 0xffu) << (8 * r);
            byte_rows[1] |= (uint64_t)(d[r] >> 8) << (8 * r);
        }
        byte_rows[0] = transpose_bits(byte_rows[0]);
        byte_rows[1] = transpose_bits(byte_rows[1]);
        const int mine = __popc(any);
        int incl = mine;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
            const int up = __shfl_up(incl, s, 64);
            if (l >= s)
                incl += up;
        }
        if (k0 > 0)
            __syncthreads();  // the totals of the pass before have been read
        if (l == 63)
            wave_total[wave] = incl;
        __syncthreads();
        int pos = cnt + incl - mine;
#pragma unroll
        for (int w = 0; w < kActiveWaves; ++w) {
            const int wt = wave_total[w];
            pos += w < wave ? wt : 0;
            cnt += wt;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t rb = (uint32_t)(byte_rows[i / 8] >> (8 * (i % 8))) & 0xffu;
            if (rb) {
                list[pos] = (uint16_t)(kt + i);
                rows[pos] = (uint8_t)rb;
                ++pos;
            }
        }
    }
    const int n_steps = (cnt + kActiveStep - 1) / kActiveStep;
    for (int e = cnt + (int)threadIdx.x; e < (n_steps + 1) * kActiveStep; e += kActiveBlock) {
        list[e] = (uint16_t)K;
        rows[e] = 0;
    }
    __syncthreads();

    const __amdgpu_buffer_rsrc_t wres = weight_resource(W, (int64_t)K * N);
    const uint32_t lane_off = n0 + 8 * c < N ? (uint32_t)(n0 + 8 * c) : kOutOfRange;  // channels past N: no request
    auto load_weights = [&](int s, u32x2 (&w)[16]) {
        const u32x4* at = reinterpret_cast<const u32x4*>(list + min(s, n_steps) * kActiveStep + 16 * q);
        const u32x4 two[2] = {at[0], at[1]};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t pair = two[i / 8][i % 8 / 2];
            const uint32_t col = i % 2 ? pair >> 16 : pair & 0xffffu;
            w[i] = __builtin_amdgcn_raw_buffer_load_b64(wres, __umul24(col, N) + lane_off, 0, NT ? 2 : 0);  // K * N < 2^31
        }
    };
    mf_i32x4 acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t)
        acc[t] = mf_i32x4{0, 0, 0, 0};
    auto products = [&](int s, const u32x2 (&w)[16]) {
        const u32x4 rb = *reinterpret_cast<const u32x4*>(rows + min(s, n_steps) * kActiveStep + 16 * q);
        mf_i32x4 a;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            a[i] = (int32_t)((rb[i] >> c) & 0x01010101u);  // rows 8 .. 15 are not stored
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t ch[4][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t r[4] = {w[4 * i][h], w[4 * i + 1][h], w[4 * i + 2][h], w[4 * i + 3][h]};
                transpose_bytes(r, ch[i]);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const mf_i32x4 bw = {(int32_t)ch[0][t], (int32_t)ch[1][t], (int32_t)ch[2][t], (int32_t)ch[3][t]};
                acc[4 * h + t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, bw, acc[4 * h + t], 0, 0, 0);
            }
        }
    };
    u32x2 w0[16], w1[16];
    load_weights(wave, w0);
    load_weights(wave + kActiveWaves, w1);
    for (int s = wave; s < n_steps; s += 2 * kActiveWaves) {
        products(s, w0);
        load_weights(s + 2 * kActiveWaves, w0);
        __builtin_amdgcn_sched_barrier(0);
        products(s + kActiveWaves, w1);
        load_weights(s + 3 * kActiveWaves, w1);
        __builtin_amdgcn_sched_barrier(0);
    }
    // Register j of lane 16 q + c is row 4 q + j: the rows below 8 are in the
    // lower half of the lanes.  The eight waves' sums go through LDS (layout as
    // in finish_column_tile), then every thread finishes four channels of one
    // of the 256 (row, channel group) pairs.
    i32x4* part = reinterpret_cast<i32x4*>(lds);  // [j][source][32 lanes][2]
    auto half_at = [](int j, int source, int lane, int h) {
        return ((j * kActiveWaves + source) * 32 + lane) * 2 + (h ^ ((lane >> 2) & 1));
    };
    __syncthreads();  // the list has been read
    if (l < 32) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                part[half_at(j, wave, l, h)] = i32x4{acc[4 * h][j], acc[4 * h + 1][j], acc[4 * h + 2][j], acc[4 * h + 3][j]};
    }
    __syncthreads();
    const int j = wave % 4, r = 4 * (l / 32) + j, c4 = l % 32;
    float* o = wave < 4 ? row_of(r) : nullptr;
    if (o && n0 + 4 * c4 < N) {
        i32x4 sum = part[half_at(j, 0, 16 * (l / 32) + c4 / 2, c4 % 2)];
#pragma unroll
        for (int s = 1; s < kActiveWaves; ++s)
            sum += part[half_at(j, s, 16 * (l / 32) + c4 / 2, c4 % 2)];
        store_channels(sum, o + n0 + 4 * c4, scale + n0 + 4 * c4);
    }
}

// Several projections of the same up to 8 rows in one launch, longest K first.
struct ActiveItems {
    const int8_t* W[kMfmaMaxItems];
    const float* scale[kMfmaMaxItems];
    int64_t mask_off[kMfmaMaxItems];  // words
    int64_t out_off[kMfmaMaxItems];   // floats
    int32_t K[kMfmaMaxItems];
};

template <bool NT>
__global__ __launch_bounds__(kActiveBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_active_items(
    const ActiveItems items, int N, int n_coltiles, const uint64_t* __restrict__ mask, int B,
    float* __restrict__ out)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const int item = blockIdx.x / n_coltiles;
    const int n0 = blockIdx.x % n_coltiles * kColChannels;
    const int K = items.K[item];
    const int pitch = (K + 63) / 64 * (int)sizeof(uint64_t);
    const __amdgpu_buffer_rsrc_t mres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint64_t*>(mask + items.mask_off[item]), 0, B * pitch, kBufferFlags);
    float* o = out + items.out_off[item];
    active_tile<NT>(items.W[item], items.scale[item], K, N, n0, mres, 0, pitch, B, lds,
                    [&](int r) -> float* { return r < B ? o + (int64_t)r * N : nullptr; });
}

}  // namespace spk
