// Block-wide exact top-k selection over keys held in LDS, with the tie rule
// "higher key first, then lower index".  Used for the gate-score keep sets
// (Sec. 4.5) and for the top-U query choice of SentryAttend (Sec. 4.4).
//
// The k-th largest key is found by a 4-pass radix select (8 bits per pass, a
// 256-bin LDS histogram per pass with integer atomics: the counts, hence the
// result, do not depend on the order of the atomics).  The kept indices are then
// emitted in ascending order from contiguous per-thread index ranges with one
// block-wide prefix sum.  Barriers and cross-lane moves are what it costs on short
// rows, so there is one barrier per pass (every wave scans the histogram for itself)
// and two around them: keep sets of 1024 channels 9.1 -> 8.2 us with the launch, 4096
// query scores 14.6 -> 12.7.
#pragma once

#include "common.hpp"

namespace sf {

constexpr int TOPK_SCRATCH = 4 * 256 + 16;      // ints of LDS scratch block_topk needs (16-byte aligned)

// Inclusive prefix sum over the 64 lanes of a wave, in registers (data-parallel primitives: shifts by 1, 2, 4 and 8 inside
// a row of 16 lanes, then the last lane of a row added to the rows behind it); six cross-lane moves through the LDS
// permute path take about 600 clocks one after the other, these about 60.
__device__ __forceinline__ int wave_incl_scan(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);      // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);      // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);      // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);      // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);      // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);      // row_bcast:31 into rows 2 and 3
    return x;
}

// Sum of one int per thread over the block; every thread gets the total.
// `red` is LDS scratch of at least NT/64 ints.
template <int NT>
__device__ __forceinline__ int block_sum(int v, int *red)
{
    v = wave_incl_scan(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = v;
    __syncthreads();
    int t = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) t += red[i];
    return t;
}

// keys[0..n) in LDS, n <= 16384; the caller's writes to it need no barrier of their own, but `scratch` must not be in
// use.  Selects the k largest (1 <= k <= n).  For every index i, in ascending order within a thread, calls
// emit(i, kept, pos) where pos is the rank of i among the kept indices (ascending index order) when kept; at that point
// keys[i] is read by nobody else any more.  `positive`: k is the number of keys > 0 (no search).  Must be called by all NT threads; `scratch` is LDS of TOPK_SCRATCH ints.
template <int NT, class Emit>
__device__ void block_topk(uint32_t *keys, int n, int k, int *scratch, bool positive, Emit emit)
{
    int *red = scratch + 4 * 256;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int j = tid; j < 4 * 256; j += NT) scratch[j] = 0;
    __syncthreads();

    // k-th largest key T, most significant byte first
    uint32_t prefix = 0, mask = 0;
    int kk = positive ? 0 : k;
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        if (positive) break;
        const int shift = 24 - 8 * pass;
        int *hist = scratch + pass * 256;
        for (int i0 = 0; i0 < n; i0 += NT) {                    // the same trip count for every lane of a wave
            const int i = i0 + tid;
            const uint32_t key = i < n ? keys[i] : 0u;
            const int bin = (int)((key >> shift) & 255u);
            bool use = i < n && (key & mask) == prefix;
            if (pass == 0) {
                // the top byte is sign and exponent: most lanes share one or two bins, and a wave's atomics on one
                // address run one after the other
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const unsigned long long left = __ballot(use);
                    if (!left) break;
                    const int src = __ffsll((long long)left) - 1;
                    const int b = __builtin_amdgcn_readlane(bin, src);
                    const unsigned long long same = __ballot(use && bin == b);
                    if (lane == src) atomicAdd(&hist[b], __popcll(same));
                    use = use && bin != b;
                }
            }
            if (use) atomicAdd(&hist[bin], 1);
        }
        __syncthreads();
        // lane owns bins 252 - 4*lane .. 255 - 4*lane (descending with the lane, so that a prefix sum runs from the top);
        // find the bin holding the kk-th largest candidate
        const int4 hv = reinterpret_cast<const int4 *>(hist)[63 - lane];
        const int h[4] = {hv.x, hv.y, hv.z, hv.w};
        const int local = h[0] + h[1] + h[2] + h[3];
        int run = wave_incl_scan(local) - local;        // candidates in strictly higher bins
        int digit = -1, rest = 0;
#pragma unroll
        for (int j = 3; j >= 0; --j) {
            if (run < kk && run + h[j] >= kk) { digit = 252 - 4 * lane + j; rest = kk - run; }
            run += h[j];
        }
        const int at = __ffsll((long long)__ballot(digit >= 0)) - 1;      // exactly one lane
        prefix |= (uint32_t)__builtin_amdgcn_readlane(digit, at) << shift;
        kk = __builtin_amdgcn_readlane(rest, at);
        mask |= 255u << shift;
    }
    const uint32_t T = prefix;
    const int need = kk;                            // how many keys == T are kept (lowest indices)

    // emit in ascending index order: thread t owns indices [t*E, (t+1)*E).  One prefix sum counts the keys above T (high
    // half) and those equal to it (low half).
    const int E = (n + NT - 1) / NT;
    const int i0 = min(n, tid * E), i1 = min(n, i0 + E);
    int c = 0;
    for (int i = i0; i < i1; ++i) { const uint32_t key = keys[i]; c += key > T ? 1 << 16 : key == T ? 1 : 0; }
    const int x = wave_incl_scan(c);
    if (lane == 63) red[w] = x;
    __syncthreads();
    int before = x - c;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) before += i < w ? red[i] : 0;
    int eqr = before & 0xffff;
    int pos = (before >> 16) + min(eqr, need);
    for (int i = i0; i < i1; ++i) {
        const uint32_t key = keys[i];
        const bool eq = key == T;
        const bool kept = key > T || (eq && eqr < need);
        eqr += eq;
        emit(i, kept, pos);
        pos += kept;
    }
}

}  // namespace sf
