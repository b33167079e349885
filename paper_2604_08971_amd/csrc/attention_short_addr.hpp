// Addresses and LDS layout of attention_short.hip, apart from the kernel so that a host program can walk them.
#pragma once

#include <cstddef>
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

// LDS: keys of the head (later the partial results of the waves) | sum of every wave's queries | selection
// keys | largest product of every query (with the keys of the score) | mask words | rows of the active queries (first the
// mask words of the key sample) | partial sums of the mean key (later
// the references of every wave's queries) | mean key | context vector (16 bits)
template <int DH, int NW>
struct ShortLds {
    size_t keys_at, ml, sel_keys, qmax, words, rows, red, kbar, ctx, bytes;
    SF_SHORT_ADDR ShortLds(int L, int U)
    {
        const size_t Lr = (size_t)(L + 31) / 32 * 32, k = Lr * DH * 2, p = (size_t)NW * 32 * DH * 4;
        keys_at = 0;
        ml = k > p ? k : p;
        sel_keys = ml + NW * 32 * 4;
        qmax = sel_keys + Lr * 4;
        words = qmax + Lr * 4;
        rows = words + (Lr / 32 + 3) / 4 * 16;           // whole 16 bytes: the context vector is read so
        red = rows + (size_t)(U > 64 ? (U + 31) / 32 * 32 : 64) * 4;
        kbar = red + NW * DH * 4;
        ctx = kbar + DH * 4;
        bytes = ctx + DH * 2;
    }
};

}  // namespace sf
