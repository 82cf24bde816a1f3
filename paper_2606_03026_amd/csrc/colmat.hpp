// Matrix-core contraction read straight from the column-major weights, for
// many spike rows against one weight matrix without a packed copy of it
// (gfx950 v_mfma_i32_16x16x64_i8).
//
// The stream's tokens that use the same weight copy are the rows of one
// batch: acc[t][n] = sum_k x[t][k] Q[n][k] with x in {0,1}.  The gather reads
// every active column once per token; here a tile of up to 64 tokens reads the
// columns that any of them activates once.  (64 while every K of the stream is at
// most 8192, 32 up to 16256, 16 beyond: kColumnMaxWords.)  Products are 0 or a
// weight and INT32 sums are exact, so the results have the gather's bits.
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
// Idle columns.  How many columns no row activates is known only on the device,
// so each workgroup decides: it stages its rows' spike words and their union,
// and counts.  Where few columns are active (list_entries) the tile walks a list
// of them, 64 to a step, with two bytes of rows per 16 tokens and column; the
// rows are looked up while the first weights are on their way.  Elsewhere, and
// in 64-row tiles, it walks all double steps and sends the loads of idle columns
// out of range, which moves no data but still costs the address unit its 16
// cycles per instruction.  9 tokens per copy on 4 copies of 44 projections (990
// MiB), rates 0.02 / 0.05 / 0.10 / 0.20 / 0.40: 52 / 88 / 129 / 168 / 188 us; all
// columns read 191 at any rate; loads sent out of range only, 106 / 122 / 143 /
// 171 / 194; the gather 45 / 99 / 175 / 324 / 619.  A list has to leave enough
// unread to pay for itself: up to 0.7 of the columns in 16-row tiles (0.1 above:
// 129 against 143 with 0.5), half of them in 32-row ones (0.05 at 24 rows 151
// against 158 with 0.7), a third of 1024 or fewer columns (8 projections of 256
// and 1024 columns at 0.1: 7.7 us against 9.1 with 0.7).  64-row tiles with a list
// would need more than half of the LDS (285 us against 212 for 64 tokens per copy).
//
// Work split.  A workgroup of 4 waves owns up to 64 tokens of one weight
// matrix and 128 channels; its waves take every fourth double step (or every
// fourth step of the list), keep two steps (16 KB) of weights in flight each,
// and add their sums through LDS, each wave finishing a quarter of the token
// rows.  (8 waves: 22 against 18 us for 9 tokens at 0.02 on 248 MiB, 65 against 69
// at 0.4; the fixed phases of a workgroup then overlap with fewer others.)  Tiles
// go longest K first, dealt to the XCDs in turn (one tile at a time: a whole
// projection at a time left some XCDs 9% more work; where rows are not whole
// 128-byte lines, a projection's tiles stay on one XCD, whose L2 serves the lines
// they share).  The token tiles of one weight tile run side by side on one XCD.
//
// Where most columns are active it is bound by HBM: 250 tokens over 4 copies of
// 44 projections (1.04 GB of weights, 68 MB of results) take 204 us, 5.4 TB/s
// (the gather 1346 us); 30 us of that are the stores (switched off in a timing
// copy), and a plain nontemporal read of 1 GiB takes 155 us.  Spike dwords read
// from global memory with each double step instead of staged in LDS, and sums
// stored 16 bytes of every 32 at a time, took 241 us.  By its counters the matrix
// units are busy for 26 us and the vector ALUs for 49, and its waves wait for
// memory 60% of their time.  Where few columns are active, it is bound by the
// phases of a workgroup (spike words, count, list, first weights, sums), about
// 12,000 cycles before and after the weights.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "buffer.hpp"
#include "bytes.hpp"
#include "gather.hpp"
#include "mfma.hpp"  // mf_i32x4

namespace spk {

constexpr int kColWaves = 4;
constexpr int kColBlock = 64 * kColWaves;
constexpr int kColChannels = 128;  // channels of a workgroup
constexpr int kColStep = 128;      // columns of a double step (two mask words)
constexpr int kColumnMaxWords = 66 * 1024;  // spike words of a tile: two workgroups on a compute unit

// The stream's projections for the matrix cores, longest K first: items are
// (weight set, projection) pairs, item i = set i % n_sets of projection proj[i / n_sets].
struct ColumnOrder {
    int32_t proj[kStreamMaxProj];
    int32_t K[kStreamMaxProj];
    int32_t mask_off[kStreamMaxProj];
};

// LDS of a workgroup: its rows' spike words, their union and the list of
// active columns, later its waves' sums.  Rows of staged words are an odd
// number of 16-byte units apart (rounded up to whole double steps), so the 16
// rows that one operand read touches lie in distinct banks.
__host__ __device__ constexpr int column_row_units(int K) { return (K + kColStep - 1) / kColStep | 1; }
__host__ __device__ constexpr int column_words(int RT, int K) { return (16 * RT * column_row_units(K) + (K + kColStep - 1) / kColStep) * 16; }
__host__ __device__ constexpr int column_round(int RT) { return RT < 2 ? RT : 2; }  // (row subtile, register) pairs of a wave's share in LDS at once

// The list form (tiles of up to 32 rows): a column takes 2 bytes of index and
// 2 RT bytes of rows, in whole steps of 64 columns and one more that is read ahead.
constexpr int kListStep = 64;
__host__ __device__ constexpr int list_entries(int RT, int K)
{
    const int most = K <= 1024 ? K / 3 : RT == 1 ? K * 7 / 10 : K / 2;
    const int want = (most + kListStep - 1) / kListStep + 1, room = (80000 - column_words(RT, K)) / (2 + 2 * RT) / kListStep;
    return RT > 2 || room < 2 ? 0 : (want < room ? want : room) * kListStep;
}
__host__ __device__ constexpr int column_lds(int RT, int K)
{
    const int words = column_words(RT, K) + list_entries(RT, K) * (2 + 2 * RT);
    const int sums = 4 * kColWaves * column_round(RT) * 2048;
    return words > sums ? words : sums;
}

// Inclusive sum over the lanes of a wave.
__device__ inline int wave_scan(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15, 31
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// Four channels' outputs: per channel one conversion (exact below 2^24, RNE
// beyond) and one binary32 multiply.
__device__ inline void store_channels(i32x4 sum, float* o, f32x4 scale)
{
    f32x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        y[e] = (float)sum[e] * scale[e];
    if ((reinterpret_cast<uintptr_t>(o) & 15) == 0) {
        __builtin_nontemporal_store(y, reinterpret_cast<f32x4*>(o));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            o[e] = y[e];
    }
}

// One step: the spike operands of the row subtiles times the weights of 8
// channels (dword 4 i + m of w holds the bytes of column i + 4 m in the order
// of the operand's bytes, four channels to a dword).
template <int RT>
__device__ __attribute__((always_inline)) inline void column_products(const mf_i32x4 (&a)[RT], const u32x2 (&w)[16],
                                                                      mf_i32x4 (&acc)[RT][8])
{
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
}

// Eight rows of 32 columns; afterwards byte b of d[i] holds the eight rows of
// column 8 b + i (four 8 x 8 bit-matrix transposes side by side, in three rounds
// of exchanged half blocks: Warren, Hacker's Delight, section 7-3).
__device__ inline void transpose_rows(uint32_t (&d)[8])
{
    auto exchange = [](uint32_t& x, uint32_t& y, int s, uint32_t low) {
        const uint32_t a = (x & low) | ((y << s) & ~low), b = ((x >> s) & low) | (y & ~low);
        x = a;
        y = b;
    };
#pragma unroll
    for (int r = 0; r < 4; ++r)
        exchange(d[r], d[r + 4], 4, 0x0f0f0f0fu);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        exchange(d[r / 2 * 4 + r % 2], d[r / 2 * 4 + r % 2 + 2], 2, 0x33333333u);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        exchange(d[2 * r], d[2 * r + 1], 1, 0x55555555u);
}

// The sums of a workgroup's waves, scaled and stored.  Register j of lane
// 16 q + c of acc[rt][t] is row 16 rt + 4 q + j, channel n0 + 8 c + t; row_of(r)
// gives row r's outputs (null: none); scale is the tile's 128 in LDS.
//
// Pair p = 4 rt + j (four rows) belongs to wave p / RT, which adds the four
// waves' sums from LDS, column_round(RT) pairs at a time.  A lane's two 16-byte
// halves (channels 8 c + 4 h ..) lie side by side, swapped in every second
// group of four lanes (no two lanes of a write share a bank); read back in
// channel order, every store instruction writes whole runs of 512 bytes of
// two rows.
template <int RT, class RowOf>
__device__ inline void finish_column_tile(const mf_i32x4 (&acc)[RT][8], int wave, int l, int n0, int N,
                                          const float* scale, uint8_t* lds, RowOf row_of)
{
    constexpr int kPairs = RT;
    constexpr int kRound = column_round(RT);
    i32x4* part = reinterpret_cast<i32x4*>(lds);  // [4 kRound places][kColWaves sources][64 lanes][2]
    auto half_at = [](int place, int source, int lane, int h) {
        return ((place * kColWaves + source) * 64 + lane) * 2 + (h ^ ((lane >> 2) & 1));
    };
#pragma unroll
    for (int p0 = 0; p0 < kPairs; p0 += kRound) {
        __syncthreads();  // what lay in LDS has been read
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int i = 0; i < kRound; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int p = w * kPairs + p0 + i, rt = p / 4, j = p % 4;
                    part[half_at(w * kRound + i, wave, l, h)] =
                        i32x4{acc[rt][4 * h][j], acc[rt][4 * h + 1][j], acc[rt][4 * h + 2][j], acc[rt][4 * h + 3][j]};
                }
        __syncthreads();
        const f32x4 s4 = *reinterpret_cast<const f32x4*>(scale + 4 * (l % 32));  // written before the barriers
        constexpr int kEach = 8 * kRound / kColWaves;  // half places of a wave
#pragma unroll
        for (int k = 0; k < kEach; ++k) {
            const int unit = wave * kEach + k, place = unit / 2, g = unit % 2;
            const int p = place / kRound * kPairs + p0 + place % kRound, rt = p / 4, j = p % 4;
            const int qr = l / 32 + 2 * g, c4 = l % 32;  // row group, group of four channels
            const int n = n0 + 4 * c4;
            float* o = row_of(16 * rt + 4 * qr + j);
            if (!o || n >= N)
                continue;
            i32x4 sum = part[half_at(place, 0, 16 * qr + c4 / 2, c4 % 2)];
#pragma unroll
            for (int s = 1; s < kColWaves; ++s)
                sum += part[half_at(place, s, 16 * qr + c4 / 2, c4 % 2)];
            store_channels(sum, o + n, s4);
        }
    }
}

// 16 RT tokens x 128 channels of one item per workgroup.  NT: weight loads
// marked nontemporal.
template <int RT, bool NT>
__global__ __launch_bounds__(kColBlock) __attribute__((amdgpu_waves_per_eu(RT == 1 ? 4 : 2))) void k_stream_mat(
    const StreamOperands* __restrict__ desc, const ColumnOrder order, int n_proj,
    int n_sets, int n_tokens, int N, int n_coltiles, int n_rowtiles, const uint64_t* __restrict__ masks,
    int mask_stride, float* __restrict__ out, int64_t out_stride)
{
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ int wave_active[kColWaves];
    __shared__ __align__(16) float scales[kColChannels];

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
    const int place = item / used_sets;
    const int proj = order.proj[place], K = order.K[place], mask_off = order.mask_off[place];
    const StreamOperands ops = desc[set * n_proj + proj];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int l = threadIdx.x % 64;
    const int q = l / 16;  // column group of the operands, row group of the result
    const int c = l % 16;  // token row of the spikes, 8-channel group of the weights and the result
    const __amdgpu_buffer_rsrc_t wres = weight_resource(ops.W, (int64_t)K * N);
    const int w_bytes = K * N;
    const int n_double = (K + kColStep - 1) / kColStep;

    const uint32_t lane_off = n0 + 8 * c < N ? (uint32_t)(n0 + 8 * c) : kOutOfRange;  // channels past N: no request
    // A column past the end of W (also of a double step past the wave's last)
    // is read at the end of the resource: zeros, without a memory request.  (A
    // scalar offset beyond that end would wrap the hardware's range check.)
    // A column that no row activates is sent past the end by its lane's offset.
    const uint32_t w_off = lane_off + (uint32_t)(32 * q * N);
    auto load_weights = [&](int d, int half, uint32_t idle, u32x2 (&w)[16]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int at = 4 * half + i + 8 * m, k = kColStep * d + at;
                w[4 * i + m] = __builtin_amdgcn_raw_buffer_load_b64(wres, w_off | ((idle << (31 - at)) & kOutOfRange),
                                                                    k < K ? k * N : w_bytes, NT ? 2 : 0);
            }
    };
    u32x2 w0[16], w1[16];
    if constexpr (RT > 2) {  // most columns are active: the first double step is asked for at once
        load_weights(wave, 0, 0u, w0);
        load_weights(wave, 1, 0u, w1);
    }

    // The rows' spike words, whole double steps of them (the last one's upper
    // word may be the next row's, whose bits meet zero weights), and their union.
    const int units = column_row_units(K);
    const uint32_t* dwords = reinterpret_cast<const uint32_t*>(lds);
    uint64_t* any_words = reinterpret_cast<uint64_t*>(lds) + 16 * RT * 2 * units;
    const uint32_t* any = reinterpret_cast<const uint32_t*>(any_words);
    const int row_words = 2 * n_double;
    const float scale = threadIdx.x < kColChannels && n0 + (int)threadIdx.x < N ? ops.scale[n0 + threadIdx.x] : 0.0f;
    for (int e = threadIdx.x; e < row_words; e += kColBlock)
        any_words[e] = 0;
    __syncthreads();
    {
        const __amdgpu_buffer_rsrc_t mres = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint64_t*>(masks), 0, n_tokens * mask_stride * (int)sizeof(uint64_t), kBufferFlags);
        uint64_t* words = reinterpret_cast<uint64_t*>(lds);
        const int total = 16 * RT * row_words;
        constexpr int kBatch = 8;
        // word e = r * row_words + at, kColBlock words on each time
        const int step_r = kColBlock / row_words, step_at = kColBlock % row_words;
        int r = threadIdx.x / row_words, at = threadIdx.x % row_words;
        for (int base = threadIdx.x; base < total; base += kBatch * kColBlock) {
            u32x2 v[kBatch];
            int to[kBatch], word[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int64_t t = (int64_t)(row0 + r) * n_sets + set;
                const bool ok = r < 16 * RT && t < n_tokens;
                v[u] = __builtin_amdgcn_raw_buffer_load_b64(
                    mres, ((uint32_t)t * (uint32_t)mask_stride + (uint32_t)(mask_off + at)) * 8u | (ok ? 0u : kOutOfRange), 0, 0);
                to[u] = r < 16 * RT ? r * 2 * units + at : -1;
                word[u] = ok ? at : -1;
                r += step_r;
                at += step_at;
                if (at >= row_words) {
                    at -= row_words;
                    ++r;
                }
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const uint64_t x = __builtin_bit_cast(uint64_t, v[u]);
                if (to[u] >= 0)
                    words[to[u]] = x;
                if (word[u] >= 0 && x != 0)
                    atomicOr(reinterpret_cast<unsigned long long*>(any_words + word[u]), x);
            }
        }
        __syncthreads();
    }

    if (threadIdx.x < kColChannels)
        scales[threadIdx.x] = scale;

    mf_i32x4 acc[RT][8];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < 8; ++t)
            acc[rt][t] = mf_i32x4{0, 0, 0, 0};

    // Active columns of the tile's rows; each thread has two dwords of 32.
    const int entries = list_entries(RT, K);
    uint32_t mine[2] = {0, 0};
    int before = 0, n_list = 0;
    if (RT <= 2 && entries > 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int left = K - 32 * ((int)threadIdx.x + i * kColBlock);
            if (left > 0)
                mine[i] = any[threadIdx.x + i * kColBlock] & (left >= 32 ? ~0u : (1u << left) - 1u);
        }
        const int n = __popc(mine[0]) + __popc(mine[1]), incl = wave_scan(n);
        if (l == 63)
            wave_active[wave] = incl;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kColWaves; ++w) {
            before += w < wave ? wave_active[w] : 0;
            n_list += wave_active[w];
        }
        before += incl - n;
    }
    if (RT <= 2 && entries > 0 && n_list <= entries - kListStep) {  // the whole workgroup
        uint8_t* rows = lds + column_words(RT, K);  // [2 RT][entries]
        uint16_t* list = reinterpret_cast<uint16_t*>(rows + 2 * RT * entries);
        const int n_steps = (n_list + kListStep - 1) / kListStep;
        int pos = before;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            for (uint32_t m = mine[i]; m != 0; m &= m - 1)
                list[pos++] = (uint16_t)(32 * ((int)threadIdx.x + i * kColBlock) + __builtin_ctz(m));
        for (int e = n_list + (int)threadIdx.x; e < (n_steps + 1) * kListStep; e += kColBlock)
            list[e] = (uint16_t)K;
        __syncthreads();
        auto load_listed = [&](int s, u32x2 (&w)[16]) {
            const u32x4* at = reinterpret_cast<const u32x4*>(list + min(s, n_steps) * kListStep + 16 * q);
            const u32x4 two[2] = {at[0], at[1]};
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t pair = two[i / 8][i % 8 / 2];
                const uint32_t col = i % 2 ? pair >> 16 : pair & 0xffffu;
                w[i] = __builtin_amdgcn_raw_buffer_load_b64(wres, col * (uint32_t)N + lane_off, 0, NT ? 2 : 0);
            }
        };
        load_listed(wave, w0);
        load_listed(wave + kColWaves, w1);
        // the listed columns' rows, while the first weights are on their way
        for (int e = threadIdx.x; e < (n_steps + 1) * kListStep; e += kColBlock) {
            const int k = list[e];
#pragma unroll
            for (int g = 0; g < 2 * RT; ++g) {
                uint32_t r8 = 0;
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    r8 |= (dwords[(8 * g + r) * units * 4 + k / 32] >> (k % 32) & 1u) << r;
                rows[g * entries + e] = (uint8_t)(k < K ? r8 : 0u);
            }
        }
        __syncthreads();
        auto products = [&](int s, const u32x2 (&w)[16]) {
            mf_i32x4 a[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const u32x4 rb = *reinterpret_cast<const u32x4*>(rows + (2 * rt + c / 8) * entries +
                                                                 min(s, n_steps) * kListStep + 16 * q);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    a[rt][i] = (int32_t)((rb[i] >> (c % 8)) & 0x01010101u);
            }
            column_products<RT>(a, w, acc);
        };
        for (int s = wave; s < n_steps; s += 2 * kColWaves) {
            products(s, w0);
            load_listed(s + 2 * kColWaves, w0);
            __builtin_amdgcn_sched_barrier(0);
            products(s + kColWaves, w1);
            load_listed(s + 3 * kColWaves, w1);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        auto read_idle = [&](int d) { return ~any[min(d, n_double - 1) * 4 + q]; };
        auto products = [&](int d, int half, const u32x2 (&w)[16]) {
            mf_i32x4 a[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const uint32_t bits = dwords[((16 * rt + c) * units + d) * 4 + q];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    a[rt][i] = (int32_t)((bits >> (4 * half + i)) & 0x01010101u);
            }
            column_products<RT>(a, w, acc);
        };
        if constexpr (RT <= 2) {
            const uint32_t idle = read_idle(wave);
            load_weights(wave, 0, idle, w0);
            load_weights(wave, 1, idle, w1);
        }
        for (int d = wave; d < n_double; d += kColWaves) {
            const uint32_t idle = read_idle(d + kColWaves);
            products(d, 0, w0);
            load_weights(d + kColWaves, 0, idle, w0);
            __builtin_amdgcn_sched_barrier(0);
            products(d, 1, w1);
            load_weights(d + kColWaves, 1, idle, w1);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    finish_column_tile<RT>(acc, wave, l, n0, N, scales, lds, [&](int r) -> float* {
        const int64_t t = (int64_t)(row0 + r) * n_sets + set;
        return t < n_tokens ? out + t * out_stride + (int64_t)proj * N : nullptr;
    });
}

// ---------------------------------------------------------------------------
// The same contraction for up to 8 rows of several projections at once: at a
// rate of 0.1 seven rows touch half the columns, one row a tenth, and the
// others' weights are not read.
//
// The union of the rows' spikes is counted; up to 5/8 of the columns (25/32 where
// the packed copy comes from HBM at every step) it becomes a list in LDS with a
// byte per column holding which rows are active there (8 x 8 bit transposes of the
// rows' bytes).  A step is 64 entries of the list, lane
// 16 q + c taking entries 16 q .. 16 q + 15: its weight loads go to those
// columns, and the spike operand of row c is bit c of the entries' row bytes, a
// shift and an AND per four columns.  Entries past the list name column K, whose
// weights read as zero.  Above that the tile reads all columns, from the packed
// copy (layout in mfma.hpp), whose 1 KB pieces stream faster than scattered
// columns.  Sums and stores are as above, but with 8 waves to a workgroup.
//
// What bounds the list is the random 128-byte reads: 7 rows of the 44-projection
// stack, 143 MB of active columns, take 38 us, of which 8 are the launch, the
// lists and the sums (a timing copy with one step per wave); 4 waves a
// workgroup take 40, and wider tiles (2 or 3 x 128 channels sharing a list)
// 44 and 50: half as many workgroups leave compute units idle.  Where the lines
// lie, with a hot twentieth of the columns, listed against packed tiles against
// a launch of packed tiles alone, which does not count first: 248 MiB, 6 rows at
// 0.2 (0.75 active) 50.4 / 53.9 / 51.7 us, 7 rows (0.79) 51.8 / 53.9 / 52, 4 rows at
// 0.4 (0.88) 60 / 54 / 51, 8 rows at 0.4 60 / 54 / 52; 110 MiB, 4 rows at 0.2 (0.61)
// 26.6 / 26.5 / 25.0, 5 rows (0.69) 28.4 / 26.6 / 25.2, 8 rows at 0.4 35 / 27 / 25; 62
// MiB, 4 rows at 0.2 18.9 / 19.5 / 18.2, 3 rows at 0.4 (0.79) 22.5 / 19.4 / 18.1; 52
// MiB, 1040 wide, 2 rows at 0.4 (0.66) 20.4 / 17.3 / 16.2.
// ---------------------------------------------------------------------------
constexpr int kActiveMaxRows = 8;
constexpr int kActiveMaxK = 64 * kMaxSliceWords;
constexpr int kActiveWaves = 8;
constexpr int kActiveBlock = 64 * kActiveWaves;
constexpr int kActiveStep = 64;
constexpr int kActiveHalf = 16 * kActiveBlock;  // columns that the threads take 16 each
static_assert(kActiveMaxK <= 2 * kActiveHalf);
// list (16-bit columns) and row bytes, padded by the step read past the end;
// later the waves' sums of the 8 rows
inline int active_lds(int K)
{
    const int entries = (K + kActiveStep - 1) / kActiveStep * kActiveStep + kActiveStep;
    return std::max(3 * entries, kActiveWaves * kActiveMaxRows * kColChannels * (int)sizeof(int32_t));
}

// One workgroup: n_rows rows (spike row r at byte mask0 + r * mask_pitch of
// the resource mres) against channels n0 .. n0 + 127 of W or its packed copy P.
// NT, NTP: loads of W, of P marked nontemporal.
template <bool NT, bool NTP, class RowOf>
__device__ __attribute__((always_inline)) inline void active_tile(const int8_t* W, const int8_t* P, const float* scale, int K,
                                                                  int N, int n0,
                                                                  __amdgpu_buffer_rsrc_t mres, uint32_t mask0,
                                                                  uint32_t mask_pitch, int n_rows, uint8_t* lds,
                                                                  RowOf row_of)
{
    __shared__ int wave_total[kActiveWaves];
    __shared__ __align__(16) float scales[kColChannels];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int l = threadIdx.x % 64;
    const int q = l / 16;  // entry group of the operands, row group of the result
    const int c = l % 16;  // row of the spikes, 8-channel group of the weights and the result
    const int entries = (K + kActiveStep - 1) / kActiveStep * kActiveStep + kActiveStep;
    uint16_t* list = reinterpret_cast<uint16_t*>(lds);
    uint8_t* rows = lds + 2 * entries;

    if (threadIdx.x < kColChannels)
        scales[threadIdx.x] = n0 + (int)threadIdx.x < N ? scale[n0 + threadIdx.x] : 0.0f;

    // The rows' spikes at this thread's columns: kt .. kt + 15, and as many from
    // kActiveHalf on (the upper halves of d).
    const int kt = 16 * (int)threadIdx.x;
    uint32_t d[kActiveMaxRows], any = 0;
#pragma unroll
    for (int r = 0; r < kActiveMaxRows; ++r) {
        const uint32_t at = mask0 + r * mask_pitch + (uint32_t)kt / 8;
        d[r] = __builtin_amdgcn_raw_buffer_load_b16(mres, r < n_rows && kt < K ? at : kOutOfRange, 0, 0);
        if (K > kActiveHalf)
            d[r] |= (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(
                        mres, r < n_rows && kActiveHalf + kt < K ? at + kActiveHalf / 8 : kOutOfRange, 0, 0) << 16;
        any |= d[r];
    }
    auto valid = [](int left) { return left >= 16 ? 0xffffu : left > 0 ? (1u << left) - 1u : 0u; };
    any &= valid(K - kt) | valid(K - kActiveHalf - kt) << 16;
    const int mine = __popc(any), incl = wave_scan(mine);
    if (l == 63)
        wave_total[wave] = incl;
    __syncthreads();
    int pos = incl - mine, cnt = 0;
#pragma unroll
    for (int w = 0; w < kActiveWaves; ++w) {
        pos += w < wave ? wave_total[w] : 0;
        cnt += wave_total[w];
    }
    mf_i32x4 acc[1][8];
#pragma unroll
    for (int t = 0; t < 8; ++t)
        acc[0][t] = mf_i32x4{0, 0, 0, 0};
    const bool listed = cnt <= (NTP ? K * 25 / 32 : K * 5 / 8);  // the whole workgroup
    if (listed) {
        transpose_rows(d);
        auto add = [&](int half) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (any >> (16 * half + i) & 1) {
                    list[pos] = (uint16_t)(kt + half * kActiveHalf + i);
                    rows[pos] = (uint8_t)(d[i % 8] >> (16 * half + i / 8 * 8));
                    ++pos;
                }
        };
        add(0);
        if (K > kActiveHalf)
            add(1);
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
        auto products = [&](int s, const u32x2 (&w)[16]) {
            const u32x4 rb = *reinterpret_cast<const u32x4*>(rows + min(s, n_steps) * kActiveStep + 16 * q);
            mf_i32x4 a[1];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                a[0][i] = (int32_t)((rb[i] >> c) & 0x01010101u);  // rows 8 .. 15 are not stored
            column_products<1>(a, w, acc);
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
    } else {
        // All columns, from the packed copy: k-step s of channel set t is 1 KB,
        // lane 16 q + c holding 16 columns of channel 16 t + c.
        const int wpr = (K + 63) / 64, sets = N / 16, set0 = n0 / 16;
        const int records = sets * wpr * kMfmaSetStepBytes;
        const __amdgpu_buffer_rsrc_t pres = weight_resource(P, records);
        auto load_packed = [&](int s, u32x4 (&w)[8], uint32_t& bits) {
#pragma unroll
            for (int t = 0; t < 8; ++t)
                w[t] = __builtin_amdgcn_raw_buffer_load_b128(
                    pres, 16 * l, s < wpr && set0 + t < sets ? ((set0 + t) * wpr + s) * kMfmaSetStepBytes : records, NTP ? 2 : 0);
            bits = __builtin_amdgcn_raw_buffer_load_b16(
                mres, c < n_rows && s < wpr ? mask0 + c * mask_pitch + 8u * s + 2u * q : kOutOfRange, 0, 0);
        };
        auto products = [&](uint32_t bits, const u32x4 (&w)[8]) {
            const mf_i32x4 a = {(int32_t)expand_nibble(bits), (int32_t)expand_nibble(bits >> 4),
                                (int32_t)expand_nibble(bits >> 8), (int32_t)expand_nibble(bits >> 12)};
#pragma unroll
            for (int t = 0; t < 8; ++t)
                acc[0][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, __builtin_bit_cast(mf_i32x4, w[t]), acc[0][t], 0, 0, 0);
        };
        u32x4 w0[8], w1[8];
        uint32_t b0, b1;
        load_packed(wave, w0, b0);
        load_packed(wave + kActiveWaves, w1, b1);
        for (int s = wave; s < wpr; s += 2 * kActiveWaves) {
            products(b0, w0);
            load_packed(s + 2 * kActiveWaves, w0, b0);
            __builtin_amdgcn_sched_barrier(0);
            products(b1, w1);
            load_packed(s + 3 * kActiveWaves, w1, b1);
            __builtin_amdgcn_sched_barrier(0);
        }
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
    if (l < 32 && !listed) {  // channel 16 t + c
        int32_t* words = reinterpret_cast<int32_t*>(part);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < 8; ++t)
                words[4 * half_at(j, wave, 16 * q + 2 * t + c / 8, c / 4 % 2) + c % 4] = acc[0][t][j];
    }
    if (l < 32 && listed) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                part[half_at(j, wave, l, h)] = i32x4{acc[0][4 * h][j], acc[0][4 * h + 1][j], acc[0][4 * h + 2][j], acc[0][4 * h + 3][j]};
    }
    __syncthreads();
    const int j = wave % 4, r = 4 * (l / 32) + j, c4 = l % 32;
    float* o = wave < 4 ? row_of(r) : nullptr;
    if (o && n0 + 4 * c4 < N) {
        i32x4 sum = part[half_at(j, 0, 16 * (l / 32) + c4 / 2, c4 % 2)];
#pragma unroll
        for (int s = 1; s < kActiveWaves; ++s)
            sum += part[half_at(j, s, 16 * (l / 32) + c4 / 2, c4 % 2)];
        store_channels(sum, o + n0 + 4 * c4, *reinterpret_cast<const f32x4*>(scales + 4 * c4));
    }
}

// Several projections of the same up to 8 rows in one launch, longest K first.
struct ActiveItems {
    const int8_t* W[kMfmaMaxItems];
    const int8_t* P[kMfmaMaxItems];   // packed copy
    const float* scale[kMfmaMaxItems];
    int64_t mask_off[kMfmaMaxItems];  // words
    int64_t out_off[kMfmaMaxItems];   // floats
    int32_t K[kMfmaMaxItems];
};

template <bool NT, bool NTP>
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
    active_tile<NT, NTP>(items.W[item], items.P[item], items.scale[item], K, N, n0, mres, 0,
                         pitch, B, lds,
                    [&](int r) -> float* { return r < B ? o + (int64_t)r * N : nullptr; });
}

}  // namespace spk
