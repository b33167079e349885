// Addresses of attention_short.hip, apart from the kernel so that a host program can walk them.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define SF_SHORT_ADDR __host__ __device__ __forceinline__
#else
#define SF_SHORT_ADDR inline
#endif

namespace sf {

// Byte offset of the 8 keys that a lane reads of row l32 of V^T (rows of ld elements, of which the first Lp, a multiple of 8,
// are there) in half p of the tile of 32 keys t; lhi: the upper half of the wave.  Chunks behind the row repeat its last one:
// their keys are masked.  The lane's half is part of what is clamped: a row may be shorter than both halves.
SF_SHORT_ADDR uint32_t short_v_off(int t, int p, int l32, int lhi, uint32_t ld, int Lp)
{
    const uint32_t at = (uint32_t)(t * 64 + p * 32 + lhi * 16), last = (uint32_t)(Lp - 8) * 2u;
    return (uint32_t)l32 * ld * 2u + (at < last ? at : last);
}

}  // namespace sf
