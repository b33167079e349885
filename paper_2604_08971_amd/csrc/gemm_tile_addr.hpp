// Addresses of the operand loads of gemm_bf16_tile.hip and gemm_bf16_rows.hip, apart from the kernels so that a host program can walk them.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define SF_ADDR __host__ __device__ __forceinline__
#else
#define SF_ADDR inline
#endif

namespace sf {

// The operands of a tile are buffers: the base is the tile's first row (behind a row map: the first row of A), the
// scalar offset of a load walks K and a lane's byte offset never changes.  The record count ends the buffer with the
// operand, so the K tail (K % 64 == 32: the last K tile is half a tile) may request bytes behind a row - those of the
// next row, never used - but none behind the operand: the hardware answers those requests with zeros.
SF_ADDR uint32_t records(int64_t rows, int64_t ld, int K)
{
    const int64_t n = ((rows - 1) * ld + K) * 2;
    return n < (int64_t)0xffffffff ? (uint32_t)n : 0xffffffffu;
}

// Byte offset of the 16 bytes that lane `lane` brings in for super-rows sr4*4 .. sr4*4+3 of a tile with `rows` rows.
// Rows beyond the edge are clamped: they only feed outputs that are never stored.
SF_ADDR uint32_t lane_off(int sr4, int lane, int rows, int64_t ld, const int32_t *rmap)
{
    const int sr = sr4 * 4 + (lane >> 4), t = (lane & 15) ^ (sr & 7);
    const int at = sr * 2 + (t >> 3), r = at < rows ? at : rows - 1;
    return (uint32_t)(rmap ? rmap[r] : r) * (uint32_t)ld * 2u + (uint32_t)(t & 7) * 16u;
}

}  // namespace sf
