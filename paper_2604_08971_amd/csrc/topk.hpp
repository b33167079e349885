// Block-wide exact top-k selection over keys held in LDS, with the tie rule
// "higher key first, then lower index".  Used for the gate-score keep sets
// (Sec. 4.5) and for the top-U query choice of SentryAttend (Sec. 4.4).
//
// The k-th largest key is found from one histogram of 512 equal steps between the smallest and the largest value: the
// step that holds it has a handful of keys, which every wave ranks for itself.  Where it has more than 64, a sample shows many
// of them in one step (equal values, an outlier that leaves the others in one step), the row is longer than 8192 and the
// key not in its tail (a step near the mean of a bell curve has too many) or the values are no finite range, a 4-pass radix
// select (8 bits per pass, a 256-bin histogram per pass) finds it.  Counts come from integer atomics in LDS: they, hence the result, do
// not depend on the order of the atomics.  The kept indices are then emitted in ascending order from contiguous
// per-thread index ranges, or from the wave's counts of the keys in registers, with one block-wide prefix sum.  Barriers,
// cross-lane moves and lanes that meet in a bin are what it costs on short rows.  us with the launch, radix passes alone / so:
// keep sets of 2048 channels 7.6 / 6.7, of two values 9.3 / 10.4, with an outlier 7.6 / 8.4; of 4096 channels 9.5 / 7.9; of
// 16384, half of them kept 27 / 29; 4096 query scores 12.1 / 9.8, 48 scores 5.0 / 4.2.
#pragma once

#include "common.hpp"
#include "value_steps.hpp"

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

// Largest value of a wave (unsigned), in every lane
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    int x = (int)v;
#define SF_MAX_DPP(ctrl, rows) x = (int)max((uint32_t)x, (uint32_t)__builtin_amdgcn_update_dpp(0, x, ctrl, rows, 0xf, false))
    SF_MAX_DPP(0x111, 0xf);
    SF_MAX_DPP(0x112, 0xf);
    SF_MAX_DPP(0x114, 0xf);
    SF_MAX_DPP(0x118, 0xf);
    SF_MAX_DPP(0x142, 0xa);
    SF_MAX_DPP(0x143, 0xc);
#undef SF_MAX_DPP
    return (uint32_t)__builtin_amdgcn_readlane(x, 63);
}

// The value of a selection key (common.hpp, sortable_key)
__device__ __forceinline__ float key_value(uint32_t key)
{
    return __uint_as_float((key & 0x80000000u) ? key & 0x7fffffffu : ~key);
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

// keys[0..n) in LDS, n <= 16384; the caller's writes to it need no barrier of their own where thread t wrote the keys t,
// t + NT, ..., but `scratch` must not be in use.  Selects the k largest (1 <= k <= n).  For every index i, in ascending order
// within a thread, calls emit(i, kept, pos) where pos is the rank of i among the kept indices (ascending index order) when
// kept; at that point keys[i] is read by nobody else any more.  `positive`: k is the number of keys > 0 (no search).  Must be
// called by all NT threads; `scratch` is LDS of TOPK_SCRATCH ints.  MAXE > 0: n <= MAXE * NT, a thread then keeps its keys in
// registers.
template <int NT, int MAXE = 0, class Emit>
__device__ void block_topk(uint32_t *keys, int n, int k, int *scratch, bool positive, Emit emit)
{
    int *red = scratch + 4 * 256;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    constexpr int BINS = 512, NWV = NT / 64;        // scratch: histogram, then 64 keys, their count, extremes of the waves
    static_assert(MAXE * NWV <= 64, "counts of the waves");
    uint32_t *list = reinterpret_cast<uint32_t *>(scratch + BINS), *ext = list + 128;
    int *n_list = scratch + BINS + 64;
    uint32_t own[MAXE > 0 ? MAXE : 1];
    if constexpr (MAXE > 0) {
#pragma unroll
        for (int e = 0; e < MAXE; ++e) own[e] = tid + e * NT < n ? keys[tid + e * NT] : 0u;
    }
    auto each = [&](auto f) {                       // f(key) for the keys of this thread
        if constexpr (MAXE > 0) {
#pragma unroll
            for (int e = 0; e < MAXE; ++e) f(own[e]);
        } else {
            for (int i = tid; i < n; i += NT) f(keys[i]);
        }
    };
    uint32_t T = 0;                                 // k-th largest key
    int need = 0;                                   // how many keys == T are kept (lowest indices)
    bool found = positive;
    const bool cut = !positive && (MAXE > 0 || n <= 8192 || k <= n / 8);
    if (cut) {
#pragma unroll
        for (int j = tid; j < BINS + 128; j += NT) scratch[j] = 0;
        uint32_t hi = 0, lo = 0;                    // lo: complement of the smallest key > 0
        each([&](uint32_t key) {
            hi = max(hi, key);
            lo = max(lo, key ? ~key : 0u);
        });
        hi = wave_max_u32(hi);
        lo = wave_max_u32(lo);
        if (lane == 0) { ext[w] = hi; ext[NWV + w] = lo; }
    }
    lds_barrier();
    if (cut) {
        uint32_t hi = 0, lo = 0;
#pragma unroll
        for (int i = 0; i < NWV; ++i) { hi = max(hi, ext[i]); lo = max(lo, ext[NWV + i]); }
        const float vlo = key_value(~lo);
        float per_unit;
        bool steps = cut_range(vlo, key_value(hi), BINS, per_unit);                    // uniform, as is all of this
        auto bin_of = [&](uint32_t key) { return step_of(key_value(key), vlo, per_unit, BINS); };
        if (steps) {
            // 64 keys, the same for every wave: where a quarter of them meet in a step the histogram would be built on one address
            const int at = n < 64 ? lane : lane * n >> 6;
            const uint32_t key = at < n ? keys[at] : 0u;
            const int bin = key ? bin_of(key) : -1;
            const unsigned long long allowed = __ballot(key != 0u);
            const int first = __builtin_amdgcn_readlane(bin, allowed ? __ffsll((long long)allowed) - 1 : 0);
            steps = __popcll(__ballot(key && bin == first)) <= 16;
        }
        if (steps) {
            each([&](uint32_t key) {
                if (key) atomicAdd(&scratch[bin_of(key)], 1);
            });
            lds_barrier();
            // lane owns bins 504 - 8 lane .. 511 - 8 lane: descending, so that a prefix sum runs from the top
            const int4 h1 = reinterpret_cast<const int4 *>(scratch)[(63 - lane) * 2], h2 = reinterpret_cast<const int4 *>(scratch)[(63 - lane) * 2 + 1];
            const int h[8] = {h1.x, h1.y, h1.z, h1.w, h2.x, h2.y, h2.z, h2.w};
            int local = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) local += h[j];
            const int incl = wave_incl_scan(local);
            // the lane with the k-th largest key; none where keys of 0 would have to be kept
            const unsigned long long hit = __ballot(incl >= k);
            if (hit) {
                const int at = __ffsll((long long)hit) - 1;
                int run = incl - local, bin = 0, rest = 0, here = 0;      // run: keys in strictly higher bins
#pragma unroll
                for (int j = 7; j >= 0; --j) {
                    const bool in = run < k && run + h[j] >= k;
                    bin = in ? BINS - 8 - 8 * lane + j : bin;
                    rest = in ? k - run : rest;
                    here = in ? h[j] : here;
                    run += h[j];
                }
                bin = __builtin_amdgcn_readlane(bin, at);
                rest = __builtin_amdgcn_readlane(rest, at);
                here = __builtin_amdgcn_readlane(here, at);
                if (here <= 64) {                   // uniform over the block: every wave has read the same histogram
                    each([&](uint32_t key) {
                        if (key && bin_of(key) == bin) list[atomicAdd(n_list, 1)] = key;
                    });
                    lds_barrier();
                    const uint32_t mine = lane < here ? list[lane] : 0u;
                    int above = 0, upto = 0;
                    for (int j = 0; j < here; ++j) {
                        const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, j);
                        above += other > mine;
                        upto += other >= mine;
                    }
                    const int t = __ffsll((long long)__ballot(lane < here && above < rest && upto >= rest)) - 1;
                    T = (uint32_t)__builtin_amdgcn_readlane((int)mine, t);
                    need = rest - __builtin_amdgcn_readlane(above, t);
                    found = true;
                }
            }
        }
    }

    if (!found) {
        // the passes count from zero, most significant byte first
        lds_barrier();
        for (int j = tid; j < 4 * 256; j += NT) scratch[j] = 0;
        lds_barrier();
        uint32_t prefix = 0, mask = 0;
        int kk = k;
#pragma unroll 1
        for (int pass = 0; pass < 4; ++pass) {
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
            lds_barrier();
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
        T = prefix;
        need = kk;
    }

    // emit in ascending index order; a count holds the keys above T in its high half and those equal to it in the low one
    if constexpr (MAXE > 0) {
        // keys e*NT + tid: the wave's counts per e, then those of the waves before it
        int before[MAXE];
#pragma unroll
        for (int e = 0; e < MAXE; ++e) {
            const bool in = tid + e * NT < n;
            const unsigned long long gt = __ballot(in && own[e] > T), eq = __ballot(in && own[e] == T);
            before[e] = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(gt >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)gt, 0u)) << 16 |
                        (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(eq >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eq, 0u));
            if (lane == 0) scratch[BINS + 128 + 64 + e * NWV + w] = __popcll(gt) << 16 | __popcll(eq);
        }
        lds_barrier();
        const int c = lane < MAXE * NWV ? scratch[BINS + 128 + 64 + lane] : 0, x = wave_incl_scan(c) - c;
        // read from x before any lane leaves: it is the lanes of the low numbers that hold the sums
#pragma unroll
        for (int e = 0; e < MAXE; ++e) before[e] += __builtin_amdgcn_readlane(x, __builtin_amdgcn_readfirstlane(e * NWV + w));
#pragma unroll
        for (int e = 0; e < MAXE; ++e) {
            const int i = tid + e * NT, eqr = before[e] & 0xffff;
            if (i < n) emit(i, own[e] > T || (own[e] == T && eqr < need), (before[e] >> 16) + min(eqr, need));
        }
    } else {
        // thread t owns indices [t*E, (t+1)*E)
        const int E = (n + NT - 1) / NT;
        const int i0 = min(n, tid * E), i1 = min(n, i0 + E);
        int c = 0;
        for (int i = i0; i < i1; ++i) { const uint32_t key = keys[i]; c += key > T ? 1 << 16 : key == T ? 1 : 0; }
        const int x = wave_incl_scan(c);
        if (lane == 63) red[w] = x;
        lds_barrier();
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
}

}  // namespace sf
