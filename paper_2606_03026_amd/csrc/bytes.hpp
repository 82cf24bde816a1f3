// Byte transposes shared by the exporter and the column-major contraction.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spk {

// 4 x 4 bytes: byte i of d[j] becomes byte j of t[i].
__device__ inline void transpose_bytes(const uint32_t (&d)[4], uint32_t (&t)[4])
{
    const uint32_t lo01 = __builtin_amdgcn_perm(d[1], d[0], 0x05010400u), hi01 = __builtin_amdgcn_perm(d[1], d[0], 0x07030602u);
    const uint32_t lo23 = __builtin_amdgcn_perm(d[3], d[2], 0x05010400u), hi23 = __builtin_amdgcn_perm(d[3], d[2], 0x07030602u);
    t[0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
    t[1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
    t[2] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
    t[3] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
}

}  // namespace spk
