// 16-bit MFMA kernels whose tile owns whole rows of the output (N = 128, 256, 384 or 512), for what a layer does with its residual
// stream: x = R + A W^T + b in fp32 and LayerNorm(x) in 16 bits in one launch, so that the LayerNorm does not read the stream again
// (gemm_rows_kernel: output projection), and the same with A = act(xn W1^T + b1) formed on the way (ffn_rows_kernel: the whole FFN).
//
// What bounds them is memory and, in the FFN, the loads into LDS.  At d 512 a row of the output projection is 2 KB of residual read, 2 KB
// of stream and 1 KB of normalised row written next to 0.8 KB of A; the FFN's hidden row, 2.5 KB written by one launch and
// read by the next, stays in LDS.  us, separate launches (with the LayerNorm) / these: 65 536 rows, N 512, K 384 111 / 86; 122 880 in
// samples of 480, K 256 193 / 138; 24 576 in samples of 384, N 256, K 192 22 / 17; FFN of 65 536 rows, d 512, 1280 channels 238 / 208; of
// 122 880, 1024 channels 408 / 338; of 65 536, d 256, 640 channels 115 / 78; of 65 536, d 128, 320 channels 56 / 35.
//
// Tile 128 x N with one workgroup of eight waves per compute unit (N 384, 512: 96 and 128 accumulator registers per lane), 64 x N with two
// (N 128, 256).  Steps of 64 of K, i.e. rows of 128 bytes: with 64-byte rows a compute unit receives 52-65 KB/us where every one
// of them loads, with 128-byte rows 75-115, since the L2 moves whole lines.
//
// Bits: products, row sums and roundings run in the order of the launches that these replace (K in slices where gemm() would slice it, a
// row as layernorm_vec_kernel adds it), so that a sample's output does not depend on which of them its batch takes.  What that costs
// against a free order: 1 % of an encoder of d 128 where K is sliced, 0.7 % of one of d 512 (128 x 512 rows, six layers 2787 / 2808 us).
#include <atomic>
#include <type_traits>

#include "gemm.hpp"
#include "gemm_tile_addr.hpp"

namespace sf {

namespace {

constexpr int N_XCD = 8, NWV = 8, WAVES_N = 4, SK = 64;             // waves 2 (rows) x 4 (columns), elements of K per step
constexpr int PIECE = 64 * SK * 2;                                  // bytes: 64 rows of a K step, one load instruction of each wave

typedef __attribute__((address_space(3))) void lds_void;

// Element offset of (row, 16-byte chunk) in a unit or in the fp32 staging area of a wave: 128-byte rows in 256-byte lines, slots permuted.
// 32 rows further is + 4096 bytes, chunk + 2 c flips bits 5 and 6 (XOR c << 5), chunk ^ 1 bit 4.
__device__ __forceinline__ int lay(int row, int chunk)
{
    const int sr = row >> 1;
    return sr * 128 + ((((row & 1) << 3) | chunk) ^ (sr & 7)) * 8;
}

// x of another lane of a row's eight (er, ec = 0 .. 7): the one next to it, the one opposite (7 - ec)
__device__ __forceinline__ float beside(float x) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xb1, 0xf, 0xf, false)); }      // quad_perm
__device__ __forceinline__ float opposite(float x) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xf, 0xf, false)); }     // row_half_mirror

// A row's sum in the order of layernorm_vec_kernel, so that both give the same bits: there lane l adds columns 8 l .. 8 l + 7 one
// after the other, then lanes 32, 16, 8, 4, 2 and 1 apart are joined.  Here column 32 wn + 128 tn + 4 ec + e is with lane ec of wave column
// wn, so that l = 16 tn + 4 wn + ec / 2: an odd lane goes on where the even one before it ends, tiles two and one apart
// follow, then wave columns two and one apart (through LDS), then lanes.
// row_part: what an odd lane holds before the wave columns are joined, of the terms x(tn, e) of column e of tile tn or (SQ) their squares.
// The contraction of a square and a sum is written out: left to the compiler it is another one here than there.
template <int TN, bool SQ, class X>
__device__ __forceinline__ float row_part(X x)
{
    float p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = x(tn, e);
        p[tn] = beside(SQ ? squares4(t) : ((t[0] + t[1]) + t[2]) + t[3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) p[tn] = SQ ? __builtin_fmaf(t[e], t[e], p[tn]) : p[tn] + t[e];
    }
    return TN == 1 ? p[0] : TN == 2 ? p[0] + p[1] : TN == 3 ? (p[0] + p[2]) + p[1] : (p[0] + p[2]) + (p[1] + p[3]);
}
// red: [row][ec / 2][wave column].  Lane ec joins the wave columns of pair (ec / 2) ^ (ec / 4), so that the opposite lane holds the pair
// two away and, after that, the lane two away the other two.
__device__ __forceinline__ float row_total(const float *red, int row, int ec)
{
    const f32x4 v = *reinterpret_cast<const f32x4 *>(red + (row * 4 + ((ec >> 1) ^ (ec >> 2))) * 4);
    float s = (v[0] + v[2]) + (v[1] + v[3]);
    s += opposite(s);
    return s + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x4e, 0xf, 0xf, false));       // quad_perm: lane ^ 2
}

// A step begins: its operands have landed, and every wave is done with the step before
__device__ __forceinline__ void next_step()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

template <int ACT>
__device__ __forceinline__ float activate(float z)
{
    if (ACT == ACT_RELU) return __int_as_float(max(__float_as_int(z), 0));
    if (ACT == ACT_GELU) return gelu_erf(z);
    return z;
}

// The row block of a workgroup and this thread's place in it
struct Place {
    int b, m0, p;                                                           // sample, first row, weight set (negative: nothing to do)
    int lane, wave, wm, wn, l32, lhi;                                       // waves 2 (rows) x 4 (columns)
};
__device__ __forceinline__ Place place(const GemmArgs &a, int bm, int tiles_m, int total_tiles, int per_xcd)
{
    Place t;
    const int w = (blockIdx.x % N_XCD) * per_xcd + blockIdx.x / N_XCD;      // an XCD walks a contiguous range of row blocks
    t.p = -1;
    if (w >= total_tiles) return t;
    t.b = w / tiles_m;
    t.m0 = (w % tiles_m) * bm;
    t.p = a.pattern_id ? __builtin_amdgcn_readfirstlane(a.pattern_id[t.b]) : 0;
    t.lane = threadIdx.x & 63;
    t.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    t.wm = t.wave / WAVES_N;
    t.wn = t.wave % WAVES_N;
    t.l32 = t.lane & 31;
    t.lhi = t.lane >> 5;
    return t;
}

// An operand as a buffer; the address is the same in every lane, which the compiler has to be told (else each load becomes a loop)
__device__ __forceinline__ auto operand(const void *base, int64_t off, uint32_t n)
{
    const uint64_t at = (uint64_t)(uintptr_t)(static_cast<const char *>(base) + off);
    const uint64_t u = (uint64_t)__builtin_amdgcn_readfirstlane((int)(at >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char *>(u), 0, __builtin_amdgcn_readfirstlane((int)n), 0x00020000);
}

// The address of k-part s of a lane's fragment; pieces start on 128 bytes
__device__ __forceinline__ const char *flip(const char *p, int s)
{
    typedef const __attribute__((address_space(3))) char lds_char;
    return (const char *)(lds_char *)((uint32_t)(uintptr_t)(lds_char *)p ^ (uint32_t)(s << 5));
}

// Products of a step: `x` and `w` are this lane's addresses in X and in the first 128 rows of W, of which the next tiles are 16 KB
// apart; acc[OFF ..) are multiplied.  The fragments of a part of 16 are read while the part before is multiplied.  A wave that issues
// loads waits for the address unit, so of the two waves of a SIMD one issues its share before its products and the other between them.
// KEEP: the fragments of X are those of the step before.
template <int G, int OFF, bool KEEP, int N, int TM, class Issue>
__device__ __forceinline__ void step_mma(f32x16 (&acc)[N][TM], h16x8 (&xf)[SK / 16][TM], const char *x, const char *w, bool early, Issue issue)
{
    constexpr int NS = SK / 16;
    h16x8 wf[2][G];
    auto read = [&](int s) {
#pragma unroll
        for (int i = 0; i < G; ++i) wf[s & 1][i] = *reinterpret_cast<const h16x8 *>(flip(w, s) + i * 2 * PIECE);
        if (!KEEP) {
#pragma unroll
            for (int t = 0; t < TM; ++t) xf[s][t] = *reinterpret_cast<const h16x8 *>(flip(x, s) + t * 4096);
        }
    };
    read(0);
    if (early) issue();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (s + 1 < NS) read(s + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < G; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[OFF + i][j] = SF_MFMA16(wf[s & 1][i], xf[s][j], acc[OFF + i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (s == 0 && !early) issue();
        __builtin_amdgcn_sched_barrier(0);
    }
}

// acc of a wave = the 16-bit values of its columns, the same for every row; tile i of 32 columns begins at v[min(c0 + 128 i, last)]
template <int TN, int TM>
__device__ __forceinline__ void start_at(f32x16 (&acc)[TN][TM], const h16 *v, int c0, int last, bool with, int lhi)
{
    // wave-uniform addresses: scalar loads, of which a lane takes its half
    typedef const __attribute__((address_space(4))) uint32_t cu32;
#pragma unroll
    for (int i = 0; i < TN; ++i) {
        cu32 *u = (cu32 *)(uintptr_t)(v + min(c0 + i * 128, last));
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                const uint32_t lo = u[q * 4 + e / 2], hi = u[q * 4 + 2 + e / 2];
                const h16x2 t = __builtin_bit_cast(h16x2, lhi ? hi : lo);
#pragma unroll
                for (int j = 0; j < TM; ++j) {
                    acc[i][j][q * 4 + e] = with ? (float)t[0] : 0.f;
                    acc[i][j][q * 4 + e + 1] = with ? (float)t[1] : 0.f;
                }
            }
    }
}

// What both kernels end with: through a private staging area into row layout, the residual added, rows to C, their LayerNorm to
// lno_y.  The workgroup's LDS is free (the caller has passed a barrier behind the last step).
template <int TM, int TN>
__device__ __forceinline__ void finish_rows(const GemmArgs &a, const Place &t, f32x16 (&acc)[TN][TM], char *smem)
{
    constexpr int BM = 64 * TM, BN = 128 * TN, JR = TM * 4;                 // JR groups of 8 rows in a wave's part of the tile
    const int er = t.lane >> 3, ec = t.lane & 7;                            // row layout: 8 lanes x 16 bytes = 32 features of a row
    const int mrow0 = t.m0 + t.wm * TM * 32, ncol0 = t.wn * 32, rows_left = a.L - mrow0 - er;
    const int64_t grow0 = (int64_t)t.b * a.L;
    // the residual of 32 columns; rows beyond the sample read the last one again (never stored)
    auto fetch_r = [&](int tn, f32x4 (&rr)[JR]) {
        const int64_t ro = (grow0 + min(mrow0 + er, a.L - 1)) * a.ldr + a.r0 + ncol0 + tn * 128 + ec * 4;
        auto at = [&](int j) { return ro + (int64_t)min(j * 8, max(rows_left - 1, 0)) * a.ldr; };
        if (!a.R) {
#pragma unroll
            for (int j = 0; j < JR; ++j) rr[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        } else if (a.r_f32) {
#pragma unroll
            for (int j = 0; j < JR; ++j) rr[j] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.R) + at(j)));
        } else {
#pragma unroll
            for (int j = 0; j < JR; ++j) {
                const h16x4 v = __builtin_nontemporal_load(reinterpret_cast<const h16x4 *>(static_cast<const h16 *>(a.R) + at(j)));
#pragma unroll
                for (int e = 0; e < 4; ++e) rr[j][e] = (float)v[e];
            }
        }
    };
    // one workgroup per compute unit: the residual is fetched a column block ahead; two hide its latency from each other
    constexpr int NR = TN > 2 ? 2 : 1;
    f32x4 rr[NR][JR];
    fetch_r(0, rr[0]);
    char *stg = smem + t.wave * (TM * 4096);
    float *red = reinterpret_cast<float *>(smem + NWV * TM * 4096);         // [2][row][16]
    const uint32_t wb = (uint32_t)lay(t.l32, t.lhi) * 2u;
    f32x4 z[TN][JR];
    const int64_t co = a.C ? (grow0 + mrow0 + er) * a.ldc + a.c0 + ncol0 + ec * 4 : 0;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        if (NR == 2 && tn + 1 < TN) fetch_r(tn + 1, rr[(tn + 1) % NR]);
        if (NR == 1 && tn) fetch_r(tn, rr[0]);
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = acc[tn][m][q * 4 + e];
                *reinterpret_cast<f32x4 *>(stg + ((wb ^ ((uint32_t)(q * 2) << 4)) + (uint32_t)m * 4096u)) = o;
            }
#pragma unroll
        for (int j = 0; j < JR; ++j) {
            f32x4 v = *reinterpret_cast<const f32x4 *>(stg + lay(j * 8 + er, ec) * 2);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += rr[tn % NR][j][e];
            z[tn][j] = v;
        }
        if (a.C && a.c_f32) {
#pragma unroll
            for (int j = 0; j < JR; ++j)
                if (j * 8 < rows_left)
                    __builtin_nontemporal_store(z[tn][j], reinterpret_cast<f32x4 *>(static_cast<float *>(a.C) + co + (int64_t)(j * 8) * a.ldc + tn * 128));
        } else if (a.C) {
#pragma unroll
            for (int j = 0; j < JR; ++j) {
                h16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (h16)z[tn][j][e];
                if (j * 8 < rows_left)
                    __builtin_nontemporal_store(o, reinterpret_cast<h16x4 *>(static_cast<h16 *>(a.C) + co + (int64_t)(j * 8) * a.ldc + tn * 128));
            }
        }
    }
    if (!a.lno_y) return;

    // ---- LayerNorm of the rows (two passes over the registers)
    const int r0 = t.wm * TM * 32 + er, slot = (ec >> 1) * 4 + t.wn;
    float mean[JR], inv[JR];
#pragma unroll
    for (int j = 0; j < JR; ++j) {
        const float s = row_part<TN, false>([&](int tn, int e) { return z[tn][j][e]; });
        if (ec & 1) red[(r0 + j * 8) * 16 + slot] = s;
    }
    lds_barrier();
#pragma unroll
    for (int j = 0; j < JR; ++j) {
        mean[j] = row_total(red, r0 + j * 8, ec) / BN;
        const float s = row_part<TN, true>([&](int tn, int e) { return z[tn][j][e] - mean[j]; });
        if (ec & 1) red[BM * 16 + (r0 + j * 8) * 16 + slot] = s;
    }
    lds_barrier();
#pragma unroll
    for (int j = 0; j < JR; ++j) inv[j] = 1.0f / sqrtf(row_total(red + BM * 16, r0 + j * 8, ec) / BN + a.lno_eps);
    h16 *yp = static_cast<h16 *>(a.lno_y) + (grow0 + mrow0 + er) * (int64_t)BN + ncol0 + ec * 4;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const h16x4 g = *reinterpret_cast<const h16x4 *>(static_cast<const h16 *>(a.lno_g) + ncol0 + tn * 128 + ec * 4);
        const h16x4 bt = *reinterpret_cast<const h16x4 *>(static_cast<const h16 *>(a.lno_b) + ncol0 + tn * 128 + ec * 4);
#pragma unroll
        for (int j = 0; j < JR; ++j) {
            float n[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) n[e] = (z[tn][j][e] - mean[j]) * inv[j];
            const h16x4 o = scale_shift(n, g, bt);
            if (j * 8 < rows_left) *reinterpret_cast<h16x4 *>(yp + (int64_t)(j * 8) * BN + tn * 128) = o;
        }
    }
}

constexpr size_t after_of(int TM) { return (size_t)NWV * TM * 4096 + 64 * TM * 16 * 2 * 4; }      // staging and row sums of finish_rows()
constexpr size_t at_least(size_t a, size_t b) { return a > b ? a : b; }

// Where gemm() would slice K over S waves (gemm_slice_kernel: wave s takes K tiles s, s + S, .. from zero, and the slices are added to
// the bias one after the other), a tile here walks K in that order too and keeps a sum per slice, so that the bits do not depend on
// which kernel runs.  S is 4 or 8, or 1: all of K in one chain that begins with the bias, as in the other kernels.
struct Slices {
    int nk, S;                                                              // K tiles, slices
    __device__ __forceinline__ bool ends(int t) const { return t + S >= nk; }
    __device__ __forceinline__ int after(int t) const { return ends(t) ? (t & (S - 1)) + 1 : t + S; }
};
template <int TN, int TM>
__device__ __forceinline__ void clear(f32x16 (&acc)[TN][TM])
{
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
}
// acc += slice, slice = 0
template <int TN, int TM>
__device__ __forceinline__ void join(f32x16 (&acc)[TN][TM], f32x16 (&slice)[TN][TM])
{
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] += slice[i][j][e];
    clear(slice);
}

// (64 * TM) x (128 * TN) tile; a wave owns 32 * TM rows of TN tiles of 32 columns, 128 apart.  Two buffers: the operands of a step
// are on their way while the step before is multiplied.
template <int TM, int TN, bool SL>
__device__ __forceinline__ void gemm_rows(const GemmArgs &a, int slices, int tiles_m, int total_tiles, int per_xcd)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BM = 64 * TM, BN = 128 * TN, BUF = (TM + 2 * TN) * PIECE;      // X, then W
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const Place t = place(a, BM, tiles_m, total_tiles, per_xcd);
    if (t.p < 0) return;
    const int nk = a.K / SK;

    const int64_t row = (int64_t)t.b * a.L + t.m0;
    const auto xr = operand(a.A, row * a.lda * 2, records((int64_t)a.B * a.L - row, a.lda, a.K));
    const auto wr = operand(a.W, (int64_t)t.p * a.w_pstride * 2, records(a.N, a.ldw, a.K));
    uint32_t xoff[TM];
#pragma unroll
    for (int j = 0; j < TM; ++j) xoff[j] = lane_off(t.wave + j * NWV, t.lane, min(BM, a.L - t.m0), a.lda, nullptr);
    const uint32_t woff = lane_off(t.wave, t.lane, 128, a.ldw, nullptr);
    auto load = [&](int k, int buf) {
        char *to = smem + buf * BUF + t.wave * 1024;
#pragma unroll
        for (int j = 0; j < TM; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void *)(to + j * PIECE), 16, xoff[j], k * (SK * 2), 0, 0);
#pragma unroll
        for (int j = 0; j < 2 * TN; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (lds_void *)(to + (TM + j) * PIECE), 16, woff, k * (SK * 2) + j * 64 * (int)a.ldw * 2, 0, 0);
    };
    load(0, 0);
    f32x16 acc[TN][TM];                                                     // [feature tile][token tile]
    start_at(acc, a.bias ? static_cast<const h16 *>(a.bias) + (int64_t)t.p * a.bias_pstride : static_cast<const h16 *>(a.W), t.wn * 32, BN - 32,
             a.bias != nullptr, t.lhi);
    const uint32_t xbase = (uint32_t)lay(t.wm * TM * 32 + t.l32, t.lhi) * 2u, wbase = (uint32_t)lay(t.wn * 32 + t.l32, t.lhi) * 2u + TM * PIECE;
    const Slices order{nk, slices};
    f32x16 slice[SL ? TN : 1][SL ? TM : 1];
    if constexpr (SL) clear(slice);
    for (int k = 0, tile = 0; k < nk; ++k) {
        next_step();
        const char *buf = smem + (k & 1) * BUF;
        const int next = SL ? order.after(tile) : k + 1;
        h16x8 xf[SK / 16][TM];
        auto issue = [&] {
            if (k + 1 < nk) load(next, (k + 1) & 1);
        };
        if constexpr (SL) {
            step_mma<TN, 0, false>(slice, xf, buf + xbase, buf + wbase, t.wm == 0, issue);
            if (order.ends(tile)) join(acc, slice);
        } else {
            step_mma<TN, 0, false>(acc, xf, buf + xbase, buf + wbase, t.wm == 0, issue);
        }
        tile = next;
    }
    next_step();
    finish_rows(a, t, acc, smem);
#endif
}
template <int TM, int TN>
__global__ __launch_bounds__(64 * NWV, TN <= 2 ? 4 : 2) void gemm_rows_kernel(GemmArgs a, int tiles_m, int total_tiles, int per_xcd)
{
    gemm_rows<TM, TN, false>(a, 1, tiles_m, total_tiles, per_xcd);
}
template <int TM, int TN>
__global__ __launch_bounds__(64 * NWV, 4) void gemm_rows_sliced_kernel(GemmArgs a, int slices, int tiles_m, int total_tiles, int per_xcd)
{
    gemm_rows<TM, TN, true>(a, slices, tiles_m, total_tiles, per_xcd);
}

// The whole FFN of a row block: H = act(xn W1^T + b1) is formed in chunks of HC hidden channels, which stay in LDS as the second
// product's operand: the hidden activations (2.5 KB a row, written and read again by two launches) never reach memory.
// SL: the bits of a sliced first product (up_sliced: at most four K tiles, each a slice) or second one (`slices` as above: the
// chunks then take the tiles of 64 channels in that order).  Chunks of two tiles only, and registers for one workgroup per compute unit:
// a problem that gemm() slices has no more tiles than that, or hardly.
struct FfnUp { const void *xn, *W1, *b1; int64_t w1_pstride, b1_pstride; int up_sliced, slices; };

constexpr int ffn_g(int TN) { return TN == 4 ? 2 : TN; }               // the second product takes 128 g columns at a time
constexpr size_t ffn_buf(int TM, int TN, int TH) { return at_least(TM + 2 * TH, 2 * ffn_g(TN)) * PIECE; }
constexpr size_t ffn_lds(int TM, int TN, int TH) { return (size_t)TM * TH * 16384 + 2 * ffn_buf(TM, TN, TH); }

template <int TM, int TN, int TH, int ACT, bool SL>
__device__ __forceinline__ void ffn_rows(const GemmArgs &a, const FfnUp &u, int tiles_m, int total_tiles, int per_xcd)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BM = 64 * TM, BN = 128 * TN, HC = 128 * TH, HT = BM * SK * 2;      // HT: bytes of 64 channels of H
    constexpr int G = ffn_g(TN), PARTS = TN / G, BUF = (int)ffn_buf(TM, TN, TH);
    extern __shared__ __attribute__((aligned(16))) char smem[];             // H [HC / 64][BM rows][128 bytes], then the ring
    const Place t = place(a, BM, tiles_m, total_tiles, per_xcd);
    if (t.p < 0) return;
    const int F = a.K;                                                      // hidden channels
    constexpr int s1 = BN / SK;                                             // steps of the first product of a chunk
    const int64_t row = (int64_t)t.b * a.L + t.m0;
    const auto xr = operand(u.xn, row * BN * 2, records((int64_t)a.B * a.L - row, BN, BN));
    const auto w1r = operand(u.W1, (int64_t)t.p * u.w1_pstride * 2, records(F, BN, BN));
    const auto w2r = operand(a.W, (int64_t)t.p * a.w_pstride * 2, records(BN, F, F));
    uint32_t xoff[TM];
#pragma unroll
    for (int j = 0; j < TM; ++j) xoff[j] = lane_off(t.wave + j * NWV, t.lane, min(BM, a.L - t.m0), BN, nullptr);
    const uint32_t w1off = lane_off(t.wave, t.lane, 128, BN, nullptr), w2off = lane_off(t.wave, t.lane, 128, F, nullptr);
    char *const bufs = smem + HC * BM * 2;
    int buf = 0;                                                            // of the step to come
    auto load1 = [&](int c0, int cb, int s, int bf) {                       // X and W1 of a step of the first product; cb: SL, the second tile
        char *to = bufs + bf * BUF + t.wave * 1024;
#pragma unroll
        for (int j = 0; j < TM; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void *)(to + j * PIECE), 16, xoff[j], s * (SK * 2), 0, 0);
#pragma unroll
        for (int j = 0; j < 2 * TH; ++j)                                    // rows behind the last channel: zeros, never used
            __builtin_amdgcn_raw_ptr_buffer_load_lds(w1r, (lds_void *)(to + (TM + j) * PIECE), 16, w1off, (SL && j ? cb : c0 + j * 64) * (BN * 2) + s * (SK * 2), 0, 0);
    };
    auto load2 = [&](int c, int part, int bf) {                             // W2 of 64 channels from c
        char *to = bufs + bf * BUF + t.wave * 1024;
#pragma unroll
        for (int j = 0; j < 2 * G; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(w2r, (lds_void *)(to + j * PIECE), 16, w2off, c * 2 + (part * G * 128 + j * 64) * F * 2, 0, 0);
    };
    static_assert(!SL || (TH == 1 && PARTS == 1), "two tiles of channels a chunk");
    const Slices order{F / SK, u.slices};
    int ca = 0, cb = SL && F > SK ? order.after(0) * SK : F;                // SL: the channels of the two tiles of a chunk (F: none)
    load1(0, cb, 0, 0);

    f32x16 acc[TN][TM], slice[SL ? TN : 1][SL ? TM : 1];
    start_at(acc, a.bias ? static_cast<const h16 *>(a.bias) + (int64_t)t.p * a.bias_pstride : static_cast<const h16 *>(a.W), t.wn * 32, BN - 32,
             a.bias != nullptr, t.lhi);
    const bool down_sliced = SL && u.slices > 1;
    if constexpr (SL) {
        clear(slice);
        if (!down_sliced) join(slice, acc);                                 // the chain begins with the bias
    }
    const uint32_t xbase = (uint32_t)lay(t.wm * TM * 32 + t.l32, t.lhi) * 2u, wbase = (uint32_t)lay(t.wn * 32 + t.l32, t.lhi) * 2u;
    // H: channels 128 i + 32 wn + 8 q + 4 lhi .. are chunk (wn & 1) * 4 + q of tile 2 i + wn / 2 of 64 channels
    const uint32_t hwrite = (uint32_t)lay(t.wm * TM * 32 + t.l32, (t.wn & 1) * 4) * 2u + t.lhi * 8u;
    for (int c0 = 0; c0 < F; c0 += HC) {
        f32x16 h[TH][TM], hs[SL ? TH : 1][SL ? TM : 1];
        // channels behind the last: any finite start, never used
        start_at(h, u.b1 ? static_cast<const h16 *>(u.b1) + (int64_t)t.p * u.b1_pstride : static_cast<const h16 *>(u.W1),
                 SL ? (t.wn < 2 ? ca + t.wn * 32 : cb + t.wn * 32 - 64) : c0 + t.wn * 32, F - 32, u.b1 != nullptr, t.lhi);
        if constexpr (SL) {
            clear(hs);
            if (!u.up_sliced) join(hs, h);
        }
        for (int s = 0; s < s1; ++s) {
            next_step();
            const char *b = bufs + buf * BUF;
            h16x8 xf[SK / 16][TM];
            auto issue = [&] {
                if (s + 1 < s1) load1(SL ? ca : c0, cb, s + 1, buf ^ 1);
                else load2(SL ? ca : c0, 0, buf ^ 1);
            };
            if constexpr (SL) {
                step_mma<TH, 0, false>(hs, xf, b + xbase, b + TM * PIECE + wbase, t.wm == 0, issue);
                if (u.up_sliced || s + 1 == s1) join(h, hs);
            } else {
                step_mma<TH, 0, false>(h, xf, b + xbase, b + TM * PIECE + wbase, t.wm == 0, issue);
            }
            buf ^= 1;
        }
        // H to LDS: every wave has passed a barrier behind its last read of the chunk before
#pragma unroll
        for (int i = 0; i < TH; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint2 pw;
                    pw.x = pack2_h16(activate<ACT>(h[i][j][q * 4]), activate<ACT>(h[i][j][q * 4 + 1]));
                    pw.y = pack2_h16(activate<ACT>(h[i][j][q * 4 + 2]), activate<ACT>(h[i][j][q * 4 + 3]));
                    *reinterpret_cast<uint2 *>(smem + (2 * i + t.wn / 2) * HT + (hwrite ^ (q << 4)) + j * 4096) = pw;
                }
        const int c1 = min(c0 + HC, F);
        const int na = SL && c1 < F ? order.after(cb / SK) * SK : c1, nb = SL && c1 + SK < F ? order.after(na / SK) * SK : F;
        for (int c = c0; c < c1; c += SK) {
            h16x8 xf[SK / 16][TM];
            auto after = [&] {                                              // what follows these 64 channels
                if (c + SK < c1) load2(SL ? cb : c + SK, 0, buf ^ 1);
                else if (c1 < F) load1(na, nb, 0, buf ^ 1);
            };
            next_step();
            const char *x = smem + (c - c0) / SK * HT + xbase;
            auto issue = [&] {
                if constexpr (PARTS == 2) load2(c, 1, buf ^ 1);
                else after();
            };
            if constexpr (SL) {
                step_mma<G, 0, false>(slice, xf, x, bufs + buf * BUF + wbase, t.wm == 0, issue);
                if (order.ends((c == c0 ? ca : cb) / SK)) join(acc, slice);
            } else {
                step_mma<G, 0, false>(acc, xf, x, bufs + buf * BUF + wbase, t.wm == 0, issue);
            }
            buf ^= 1;
            if constexpr (PARTS == 2) {                                     // the same channels, the other columns
                next_step();
                step_mma<G, TN - G, true>(acc, xf, x, bufs + buf * BUF + wbase, t.wm == 0, after);
                buf ^= 1;
            }
        }
        ca = na;
        cb = nb;
    }
    next_step();
    finish_rows(a, t, acc, smem);
#endif
}
template <int TM, int TN, int TH, int ACT>
__global__ __launch_bounds__(64 * NWV, TH == 2 ? 2 : 4) void ffn_rows_kernel(GemmArgs a, FfnUp u, int tiles_m, int total_tiles, int per_xcd)
{
    ffn_rows<TM, TN, TH, ACT, false>(a, u, tiles_m, total_tiles, per_xcd);
}
template <int TM, int TN, int TH, int ACT>
__global__ __launch_bounds__(64 * NWV, TN == 2 ? 2 : 4) void ffn_rows_sliced_kernel(GemmArgs a, FfnUp u, int tiles_m, int total_tiles, int per_xcd)
{
    ffn_rows<TM, TN, TH, ACT, true>(a, u, tiles_m, total_tiles, per_xcd);
}

template <class Kern, class... Extra>
int32_t launch(Kern kern, std::atomic<bool> &attr_set, size_t lds, int bm, const GemmArgs &a, hipStream_t st, Extra... extra)
{
    if (!attr_set) {                                      // setting the attribute twice is harmless
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return fail(SF_ERR_HIP, "gemm: cannot reserve %zu bytes of LDS", lds);
        attr_set = true;
    }
    const int tiles_m = ceil_div(a.L, bm), total = a.B * tiles_m, per_xcd = ceil_div(total, N_XCD);
    ProfScope prof(SF_KERNEL_GEMM, st);
    hipLaunchKernelGGL(kern, dim3(per_xcd * N_XCD), dim3(64 * NWV), lds, st, a, extra..., tiles_m, total, per_xcd);
    return SF_OK;
}

template <int TM, int TN, bool SL>
int32_t launch_rows(const GemmArgs &a, int slices, hipStream_t st)
{
    static std::atomic<bool> set{false};
    constexpr size_t lds = at_least((size_t)2 * (TM + 2 * TN) * PIECE, after_of(TM));
    if constexpr (SL) return launch(gemm_rows_sliced_kernel<TM, TN>, set, lds, 64 * TM, a, st, slices);
    else return launch(gemm_rows_kernel<TM, TN>, set, lds, 64 * TM, a, st);
}

template <int TM, int TN, int TH, int ACT, bool SL>
int32_t launch_ffn(const GemmArgs &a, const FfnUp &u, hipStream_t st)
{
    static std::atomic<bool> set{false};
    constexpr size_t lds = at_least(ffn_lds(TM, TN, TH), after_of(TM));
    if constexpr (SL) return launch(ffn_rows_sliced_kernel<TM, TN, TH, ACT>, set, lds, 64 * TM, a, st, u);
    else return launch(ffn_rows_kernel<TM, TN, TH, ACT>, set, lds, 64 * TM, a, st, u);
}

template <int ACT>
int32_t launch_ffn_act(const GemmArgs &a, const FfnUp &u, hipStream_t st)
{
    const bool sliced = u.up_sliced || u.slices > 1;
    switch (a.N / 128) {
    case 1: return sliced ? launch_ffn<1, 1, 1, ACT, true>(a, u, st) : launch_ffn<1, 1, 1, ACT, false>(a, u, st);
    case 2: return sliced ? launch_ffn<1, 2, 1, ACT, true>(a, u, st) : launch_ffn<1, 2, 1, ACT, false>(a, u, st);
    case 3: return launch_ffn<2, 3, 2, ACT, false>(a, u, st);
    default: return launch_ffn<2, 4, 2, ACT, false>(a, u, st);
    }
}

// K slices of the kernel that gemm() takes; 1: one chain
int slices_of(GemmKind kind) { return kind == GEMM_SLICE8 ? 8 : kind == GEMM_SLICE4 ? 4 : 1; }

}  // namespace

bool gemm_bf16_rows_eligible(const GemmArgs &a)
{
    if (a.epi != EPI_ROWMAJOR || a.act != ACT_NONE || a.VT || a.row_map || a.n_lim || a.k_lim || a.ln_g || a.n0) return false;
    if (a.N % 128 || a.N > 512 || a.K % SK || a.K < SK || a.lda % 8 || a.ldw % 8 || a.ldr % 4 || a.r0 % 4 || a.ldc % 4 || a.c0 % 4) return false;
    // whole aligned chunks: 16 bytes of the operands, the residual and the stream, 8 of 16-bit rows, 4 of the bias
    if (((uintptr_t)a.A | (uintptr_t)a.W | (a.r_f32 ? (uintptr_t)a.R : 0) | (a.c_f32 ? (uintptr_t)a.C : 0)) & 15) return false;
    if (((uintptr_t)a.R | (uintptr_t)a.C) & 7) return false;
    // layernorm() takes rows off their 16 bytes by a kernel that adds in another order
    if (((uintptr_t)a.lno_g | (uintptr_t)a.lno_b | (uintptr_t)a.lno_y) & 15) return false;
    if (((uintptr_t)a.bias & 3) || a.bias_pstride % 2) return false;
    return a.lda < ((int64_t)1 << 23) && a.ldw < ((int64_t)1 << 20);        // 32-bit byte offsets within a tile
}

// kind: the kernel that gemm() takes without the LayerNorm
int32_t gemm_bf16_rows(const GemmArgs &a, GemmKind kind, hipStream_t st)
{
    const int slices = slices_of(kind);
    switch (a.N / 128) {
    case 1: return slices > 1 ? launch_rows<1, 1, true>(a, slices, st) : launch_rows<1, 1, false>(a, 1, st);
    case 2: return slices > 1 ? launch_rows<1, 2, true>(a, slices, st) : launch_rows<1, 2, false>(a, 1, st);
    case 3: return launch_rows<2, 3, false>(a, 1, st);
    default: return launch_rows<2, 4, false>(a, 1, st);
    }
}

// up: the first product (A = xn), down: the second, as gemm() would take them one after the other
bool ffn_bf16_rows_eligible(const GemmArgs &up, const GemmArgs &down)
{
    if (!gemm_bf16_rows_eligible(down) || up.ln_g || up.N % 64 || up.K != down.N || up.lda != up.K || up.ldw != up.K || down.ldw != up.N) return false;
    if ((((uintptr_t)up.A | (uintptr_t)up.W) & 15) || ((uintptr_t)up.bias & 3) || up.bias_pstride % 2) return false;
    return (int64_t)up.N * up.K * 2 < ((int64_t)1 << 31);
}

int32_t ffn_bf16_rows(const GemmArgs &up, GemmKind up_kind, const GemmArgs &down, GemmKind down_kind, hipStream_t st)
{
    const FfnUp u{up.A, up.W, up.bias, up.w_pstride, up.bias_pstride, slices_of(up_kind) > 1, slices_of(down_kind)};
    return up.act == ACT_GELU ? launch_ffn_act<ACT_GELU>(down, u, st) : launch_ffn_act<ACT_RELU>(down, u, st);
}

}  // namespace sf
