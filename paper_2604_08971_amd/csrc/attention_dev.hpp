// Device helpers shared by the 16-bit attention kernels.
#pragma once

#include "common.hpp"

namespace sf {

constexpr int PAD = 8;            // 16-bit elements of row padding (16 bytes) against bank conflicts
constexpr float LOG2E = 1.4426950408889634f;
constexpr float RESCALE_LOG2 = 8.0f;    // slack of the softmax reference below the running maximum, in powers of two

// Bit j%32 of word j/32 = key j of sample b is allowed (0 beyond L).
__device__ __forceinline__ void build_mask_words(const uint8_t *kv, int L, uint32_t *words, int nwords)
{
    // one position per lane, the words from the wave's ballot: a single round of byte loads for the whole block
    // (a lane that assembled a word by itself paid 32 loads one after the other)
    const int lane = threadIdx.x & 63;
    for (int j0 = 0; j0 < nwords * 32; j0 += (int)blockDim.x) {      // the same trip count for every wave
        const int j = j0 + (int)threadIdx.x;
        const bool ok = j < L && (!kv || kv[j]);
        const unsigned long long bal = __ballot(ok);
        const int w = j >> 5;
        if ((lane & 31) == 0 && w < nwords) words[w] = (uint32_t)(bal >> (lane & 32));
    }
}

// v_permlane32_swap exchanges lanes 32..63 of its first operand with lanes 0..31 of its second: fed the same value
// twice, lane l then holds v[l % 32] in the first result and v[32 + l % 32] in the second - the values of the two
// lanes that share a query.
__device__ __forceinline__ float both_halves_max(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float both_halves_sum(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

}  // namespace sf
