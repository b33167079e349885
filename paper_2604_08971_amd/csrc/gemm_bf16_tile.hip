// bf16 MFMA GEMMs for the launches that do not fill the chip with the 256 x 256 tiles of gemm_bf16_ws.hip (see
// gemm_bf16.hip for the role of the GEMM and gemm.hpp for the arguments): short batches, short or ragged samples,
// narrow outputs.  Two kernels share loads, layout and argument handling:
//
//  * gemm_pipe_kernel: 128 x 128 tiles, four waves of 64 x 64, two workgroups per compute unit (64 KB of LDS each), so
//    that one workgroup's epilogue runs under the other's K loop.  What bounds it is LDS: a 64 x 64 wave tile reads
//    16 KB of fragments per 16 MFMAs, a K tile of a workgroup moves 96 KB through the LDS (768 clocks at 128 B/clk)
//    for 512 clocks of matrix work, which is why the 256 x 256 kernel (wave tiles of 128 x 64) stays ahead wherever
//    its tiles fill the chip.  The K loop is software-pipelined by hand: fragments are read two k-steps ahead, also
//    across the barrier, which therefore sits in the middle of a K tile - there every fragment of the tile is in
//    registers, so the tile's own slot is free for the loads of the tile after next, and the next tile must have
//    landed.  (The compiler's own order waits for the fragments right before their MFMAs: 10-15 % slower.)  Three or
//    four ring slots with one workgroup per compute unit were slower everywhere (15-40 %).
//  * gemm_slice_kernel: K sliced over the waves of a workgroup, for problems with a tile or two per compute unit: every
//    wave owns the whole tile and every NWK-th K tile in an LDS region of its own, so there is no barrier and no wait
//    on another wave until the partial tiles are summed through LDS.  Latency is all there is: 20 K tiles are
//    20 dependent steps of 0.5 us for the pipelined kernel and three for eight slices.
//
// Measured (bf16, us; 256 x 256 kernel / pipe / slice): 512 rows, N 512, K 1280, fp32 residual 32.1 / 14.3 / 6.0;
// 4096 rows, N 1280, K 512, ReLU 16.4 / 11.9 / 31.6; 24576 rows in samples of 384, N 256, K 192, residual
// 24.8 / 12.6 / 37; 37777 rows in samples of 1021, N 384, K 960 77 / 47 / 112; 65536 rows, N 2176, K 768
// 229 / 288 / 1109.
#include <algorithm>
#include <atomic>

#include "gemm.hpp"
#include "gemm_tile_addr.hpp"

namespace sf {

namespace {

constexpr int TBK = 64;                 // elements of K per ring slot
constexpr int N_XCD = 8;

typedef __attribute__((address_space(3))) void lds_void;
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Element offset of (row, 16-byte chunk) in a [rows][64] tile: 256-byte super-rows of two rows, slot XOR super-row, so
// that any 16 consecutive rows of one chunk fall into different LDS slots (16 lanes of a ds_read_b128 per cycle).
__device__ __forceinline__ int lay(int row, int chunk)
{
    const int sr = row >> 1;
    return sr * 128 + ((((row & 1) << 3) | chunk) ^ (sr & 7)) * 8;
}

template <int ACT>
__device__ __forceinline__ float activate(float z)
{
    // integer max on the bit pattern: one instruction, -0 and negatives give +0
    if (ACT == ACT_RELU) return __int_as_float(max(__float_as_int(z), 0));
    if (ACT == ACT_GELU) return gelu_erf(z);
    return z;
}

// The output tile of a workgroup.  Tiles are numbered N fastest and each XCD walks a contiguous range of them, so
// that the workgroups of an XCD share activation rows and weight tiles in its L2.
struct Tile { int b, m0, nt0, N, p; bool vt; };

__device__ __forceinline__ bool find_tile(const GemmArgs &a, int bm, int bn, int tiles_m, int tiles_n, int total, int per_xcd,
                                          Tile &t)
{
    int w = (blockIdx.x % N_XCD) * per_xcd + blockIdx.x / N_XCD;
    if (a.xcd_rows) {
        // rows of tiles of unequal cost: dealt to the XCDs round-robin
        const int s = blockIdx.x / N_XCD;
        w = ((s / tiles_n) * N_XCD + blockIdx.x % N_XCD) * tiles_n + s % tiles_n;
    }
    if (w >= total) return false;
    const int tn_i = w % tiles_n, tm_i = w / tiles_n;
    t.b = tm_i / tiles_m;
    t.m0 = (tm_i % tiles_m) * bm;
    t.p = a.pattern_id ? a.pattern_id[t.b] : 0;
    if (t.p < 0) return false;                                     // sample not in use
    t.vt = false;
    t.nt0 = tn_i * bn;
    t.N = a.n_lim ? min(a.N, a.n_lim[t.p]) : a.N;
    if (a.VT) {
        // two column ranges, each with its own tiles: [0, vt_from) row-major, [vt_from, N) transposed
        const int ta = (a.vt_from + bn - 1) / bn;
        t.vt = tn_i >= ta;
        t.nt0 = t.vt ? a.vt_from + (tn_i - ta) * bn : tn_i * bn;
        t.N = t.vt ? a.N : a.vt_from;
    }
    return t.nt0 < t.N;
}

// The operands of a tile (gemm_tile_addr.hpp)
struct Source { const char *x, *w; uint32_t nx, nw; };

__device__ __forceinline__ Source sources(const GemmArgs &a, const Tile &t)
{
    Source s;
    const int64_t row = (int64_t)t.b * a.L + t.m0;
    s.x = static_cast<const char *>(a.A) + (a.row_map ? (int64_t)0 : row * a.lda * 2);
    s.nx = records(a.row_map ? a.a_rows : (int64_t)a.B * a.L - row, a.lda, a.K);
    s.w = static_cast<const char *>(a.W) + ((int64_t)t.p * a.w_pstride + (int64_t)(a.n0 + t.nt0) * a.ldw) * 2;
    s.nw = records(a.N - t.nt0, a.ldw, a.K);
    return s;
}

template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// a bare barrier: __syncthreads() would wait for every load in flight
__device__ __forceinline__ void barrier()
{
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ------------------------------------------------------------------------------------------------- pipelined tiles
template <int ACT>
__global__ __launch_bounds__(256, 2)
void gemm_pipe_kernel(GemmArgs a, int tiles_m, int tiles_n, int total_tiles, int per_xcd)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BM = 128, BN = 128, NW = 4;
    constexpr int LX = BM / 8 / NW, LW = BN / 8 / NW, LPW = LX + LW;       // load instructions per wave and K tile
    constexpr int STAGE = (BM + BN) * TBK * 2;                             // bytes per ring slot
    extern __shared__ __attribute__((aligned(16))) char smem[];            // [2][X rows | W rows][128 bytes]

    Tile tl;
    if (!find_tile(a, BM, BN, tiles_m, tiles_n, total_tiles, per_xcd, tl)) return;
    const bool vt = tl.vt;
    const int N = tl.N, K = a.k_lim ? min(a.K, a.k_lim[tl.p]) : a.K;
    const int nk = K / TBK, nkt = (K + TBK - 1) / TBK;                     // whole K tiles, K tiles with the tail

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lhi = lane >> 5;

    const Source src = sources(a, tl);
    const auto xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(src.x), 0, (int)src.nx, 0x00020000);
    const auto wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(src.w), 0, (int)src.nw, 0x00020000);
    uint32_t xoff[LX], woff[LW];
    {
        const int32_t *rmap = a.row_map ? a.row_map + (int64_t)tl.b * a.L + tl.m0 : nullptr;
        const int rows_x = min(BM, a.L - tl.m0), rows_w = min(BN, N - tl.nt0);
#pragma unroll
        for (int j = 0; j < LX; ++j) xoff[j] = lane_off(wave + j * NW, lane, rows_x, a.lda, rmap);
#pragma unroll
        for (int j = 0; j < LW; ++j) woff[j] = lane_off(wave + j * NW, lane, rows_w, a.ldw, nullptr);
    }
    auto issue = [&](int j, int kt, int slot) {
        char *base = smem + slot * STAGE;
        if (j < LX)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void *)(base + (wave + j * NW) * 1024), 16,
                                                     xoff[j < LX ? j : 0], kt * (TBK * 2), 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (lds_void *)(base + BM * 128 + (wave + (j - LX) * NW) * 1024), 16,
                                                     woff[j < LX ? 0 : j - LX], kt * (TBK * 2), 0, 0);
    };
#pragma unroll
    for (int t = 0; t < 2; ++t)
        if (t < nkt) {
#pragma unroll
            for (int j = 0; j < LPW; ++j) issue(j, t, t);
        }

    // The accumulators start at the bias.  acc[i][j]: "A"-side tile i, "B"-side tile j; the A side are the features and
    // the B side the tokens, exchanged for the transposed range, so that a staged row below is always a B-side row.
    f32x16 acc[2][2];
    {
        const h16 *bias = a.bias ? static_cast<const h16 *>(a.bias) + (int64_t)tl.p * a.bias_pstride + a.n0 : nullptr;
        if (vt) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float f = bias ? (float)bias[min(tl.nt0 + wn * 64 + j * 32 + l32, N - 1)] : 0.f;   // clamped: never stored
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[0][j][e] = acc[1][j][e] = f;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    h16x4 bv = {};
                    if (bias) bv = *reinterpret_cast<const h16x4 *>(bias + min(tl.nt0 + wn * 64 + i * 32 + q * 8 + lhi * 4, N - 4));
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][0][q * 4 + e] = acc[i][1][q * 4 + e] = (float)bv[e];
                }
        }
    }

    // Byte addresses of this lane's fragments in a slot: tile t adds t * 4096 bytes, k-step s flips bits 5..6
    const uint32_t abase = (uint32_t)lay((vt ? wm * 64 : BM + wn * 64) + l32, lhi) * 2u;
    const uint32_t bbase = (uint32_t)lay((vt ? BM + wn * 64 : wm * 64) + l32, lhi) * 2u;
    h16x8 af[4][2], bf[4][2];
    auto read = [&](int s, int c, uint32_t slotb) {             // fragment c of k-step s: A0 B0 A1 B1
        const uint32_t base = ((c & 1) ? bbase : abase) + slotb;
        const h16x8 v = *reinterpret_cast<const h16x8 *>(smem + ((base ^ ((uint32_t)s << 5)) + (uint32_t)(c >> 1) * 4096u));
        if (c & 1) bf[s][c >> 1] = v;
        else af[s][c >> 1] = v;
    };
    if (nkt > 1) wait_vmcnt<LPW>();
    else wait_vmcnt<0>();
    barrier();
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) read(s, c, 0);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t slotb = 0;
    for (int kt = 0; kt < nk; ++kt) {
        const bool more = kt + 2 < nkt;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s == 2) {
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
                barrier();
            }
            const uint32_t rs = s < 2 ? slotb : slotb ^ (uint32_t)STAGE;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                acc[c & 1][c >> 1] = SF_MFMA16(af[s][c & 1], bf[s][c >> 1], acc[c & 1][c >> 1], 0, 0, 0);
                read((s + 2) & 3, c, rs);
                __builtin_amdgcn_sched_barrier(0);              // keep this order: MFMA, read
            }
            if (s >= 2 && more) {
#pragma unroll
                for (int j = 0; j < LPW / 2; ++j) issue((s - 2) * (LPW / 2) + j, kt + 2, slotb ? 1 : 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        slotb ^= (uint32_t)STAGE;
    }
    if (nkt > nk) {                                             // K % 64 == 32: two more k-steps, already in registers
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c & 1][c >> 1] = SF_MFMA16(af[s][c & 1], bf[s][c >> 1], acc[c & 1][c >> 1], 0, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    barrier();

    // ---- epilogue: a private 8 KB staging area per wave (64 rows of 128 bytes), whole rows to memory
    char *stg = smem + wave * 8192;
    const int64_t grow0 = (int64_t)tl.b * a.L;
    const int mrow0 = tl.m0 + wm * 64, ncol0 = tl.nt0 + wn * 64;
    const int er = lane >> 3, ec = lane & 7;                    // 8 lanes x 16 bytes = one row, 8 rows per instruction
    if (vt || (!a.c_f32 && !a.R)) {
        // 4 consecutive A-side values of a lane are one 8-byte LDS write; the chunk index only flips address bits 4..6
        const uint32_t wbase = (uint32_t)lay(l32, 0) * 2u + (uint32_t)lhi * 8u;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float z = acc[i][j][q * 4 + e];
                        v[e] = ACT == ACT_RELU ? z : activate<ACT>(z);
                    }
                    uint2 pw;
                    pw.x = pack2_h16(v[0], v[1]);
                    pw.y = pack2_h16(v[2], v[3]);
                    i16x4 m = __builtin_bit_cast(i16x4, pw);
                    if (ACT == ACT_RELU) {                      // on the rounded values: rounding never changes the sign
                        const i16x4 z = {0, 0, 0, 0};
                        m = __builtin_elementwise_max(m, z);
                    }
                    *reinterpret_cast<uint2 *>(stg + ((wbase ^ ((uint32_t)(i * 4 + q) << 4)) + (uint32_t)j * 4096u)) =
                        __builtin_bit_cast(uint2, m);
                }
        if (vt) {
            h16 *V = static_cast<h16 *>(a.VT) + (int64_t)tl.b * a.vt_b;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const h16x8 o = *reinterpret_cast<const h16x8 *>(stg + lay(j * 8 + er, ec) * 2);
                const int n = ncol0 + j * 8 + er, i = mrow0 + ec * 8;
                h16 *dst = V + (int64_t)(n - a.vt_from) * a.vt_n + i;
                if (n < N && i + 7 < a.L) {
                    *reinterpret_cast<h16x8 *>(dst) = o;
                } else if (n < N) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (i + e < a.L) dst[e] = o[e];
                }
            }
        } else {
            h16 *cp = static_cast<h16 *>(a.C) + (grow0 + mrow0 + er) * a.ldc + a.c0 + ncol0 + ec * 8;
            const bool col_ok = ncol0 + ec * 8 < N;             // N % 8 == 0: a chunk is all in or all out
            const int rows_left = a.L - mrow0 - er;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const h16x8 o = *reinterpret_cast<const h16x8 *>(stg + lay(j * 8 + er, ec) * 2);
                if (col_ok && j * 8 < rows_left) *reinterpret_cast<h16x8 *>(cp + (int64_t)(j * 8) * a.ldc) = o;
            }
        }
        return;
    }
    // residual and / or fp32 output: 64 tokens x 32 features of fp32 at a time; the residual of a pass is read before the
    // staging, so its latency is paid once per pass
    const uint32_t wbase32 = (uint32_t)lay(l32, lhi) * 2u;
    const int rows_left = a.L - mrow0 - er;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int n = ncol0 + i * 32 + ec * 4;
        const bool col_ok = n < N;
        const int64_t co0 = (grow0 + mrow0 + er) * a.ldc + a.c0 + n;
        const int64_t ro0 = (grow0 + min(mrow0 + er, a.L - 1)) * a.ldr + a.r0 + min(n, N - 4);     // clamped: never stored
        auto rrow = [&](int j) { return ro0 + (int64_t)min(j * 8, max(rows_left - 1, 0)) * a.ldr; };
        f32x4 rr[8];
        if (a.R && a.r_f32) {
#pragma unroll
            for (int j = 0; j < 8; ++j) rr[j] = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.R) + rrow(j));
        } else if (a.R) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const h16x4 t = *reinterpret_cast<const h16x4 *>(static_cast<const h16 *>(a.R) + rrow(j));
#pragma unroll
                for (int e = 0; e < 4; ++e) rr[j][e] = (float)t[e];
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = activate<ACT>(acc[i][j][q * 4 + e]);
                *reinterpret_cast<f32x4 *>(stg + ((wbase32 ^ ((uint32_t)(q * 2) << 4)) + (uint32_t)j * 4096u)) = o;
            }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            f32x4 v = *reinterpret_cast<const f32x4 *>(stg + lay(j * 8 + er, ec) * 2);
            if (a.R) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += rr[j][e];
            }
            if (col_ok && j * 8 < rows_left) {
                const int64_t co = co0 + (int64_t)(j * 8) * a.ldc;
                if (a.c_f32) {
                    *reinterpret_cast<f32x4 *>(static_cast<float *>(a.C) + co) = v;
                } else {
                    h16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = (h16)v[e];
                    *reinterpret_cast<h16x4 *>(static_cast<h16 *>(a.C) + co) = o;
                }
            }
        }
    }
#endif
}

// ----------------------------------------------------------------------------------------------------- K slices
// Sum over the eight lanes 8 i .. 8 i + 7, in each of them
__device__ __forceinline__ float sum8(float x)
{
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xb1, 0xf, 0xf, false));      // quad_perm: lane ^ 1
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4e, 0xf, 0xf, false));      // quad_perm: lane ^ 2
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xf, 0xf, false));      // row_half_mirror: lane 7 - i
}

// (TM * 32) x (TN * 32) tile; wave w takes the K tiles w, w + NWK, ... through its own LDS region.
// LN: the rows of A come unnormalised, in fp32 (1) or 16 bits (2), and at most two K tiles of 64 per wave.  A wave then holds
// its K tiles of the rows in registers, the waves exchange mean and squared deviations of their 64 columns (joined as in a
// parallel variance: no less exact than two passes over the row), and the normalised rows go to LDS.  Every column of tiles
// does that again for its rows, which costs 0.7 us where the launch of a LayerNorm is 3 to 4.
template <int TM, int TN, int NWK, int ACT, int LN>
__global__ __launch_bounds__(64 * NWK)
void gemm_slice_kernel(GemmArgs a, int tiles_m, int tiles_n, int total_tiles, int per_xcd)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BM = TM * 32, BN = TN * 32, LX = BM / 8, LW = BN / 8, BUF = (BM + BN) * TBK * 2;     // bytes
    extern __shared__ __attribute__((aligned(16))) char smem[];
    Tile tl;
    if (!find_tile(a, BM, BN, tiles_m, tiles_n, total_tiles, per_xcd, tl)) return;
    const int N = tl.N, K = a.k_lim ? min(a.K, a.k_lim[tl.p]) : a.K;
    const int nkt = (K + TBK - 1) / TBK;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    char *mine = smem + wave * BUF;

    const Source src = sources(a, tl);
    const auto xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(src.x), 0, (int)src.nx, 0x00020000);
    const auto wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(src.w), 0, (int)src.nw, 0x00020000);
    uint32_t xoff[LX], woff[LW];
    {
        const int32_t *rmap = a.row_map ? a.row_map + (int64_t)tl.b * a.L + tl.m0 : nullptr;
        const int rows_x = min(BM, a.L - tl.m0), rows_w = min(BN, N - tl.nt0);
#pragma unroll
        for (int j = 0; j < LX; ++j) xoff[j] = lane_off(j, lane, rows_x, a.lda, rmap);
#pragma unroll
        for (int j = 0; j < LW; ++j) woff[j] = lane_off(j, lane, rows_w, a.ldw, nullptr);
    }
    f32x16 acc[TN][TM];                                         // [feature tile][token tile]
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // What the epilogue adds: bias and residual of the thread's outputs.  With one output chunk per thread (the 32 x 64 tile) it is
    // on its way with the first K tiles, since read at the end it is a memory round trip of its own; four chunks would cost
    // the 64 x 64 tile more in registers than that.
    constexpr int NT = 64 * NWK, CPR = BN / 4, NC = BM * CPR / NT;
    static_assert(NC * NT == BM * CPR, "whole chunks per thread");
    const h16 *bias = a.bias ? static_cast<const h16 *>(a.bias) + (int64_t)tl.p * a.bias_pstride + a.n0 : nullptr;
    struct Added { h16x4 bias; u32x4 res; };                    // res: fp32, or 16 bits in the first two words
    auto fetch_added = [&](int c) {
        const int i = tl.m0 + c / CPR, n = tl.nt0 + c % CPR * 4;
        Added x{};
        if (tl.vt || i >= a.L || n >= N) return x;
        if (bias) x.bias = *reinterpret_cast<const h16x4 *>(bias + n);
        if (!a.R) return x;
        const int64_t ro = ((int64_t)tl.b * a.L + i) * a.ldr + a.r0 + n;
        if (a.r_f32) {
            x.res = *reinterpret_cast<const u32x4 *>(static_cast<const float *>(a.R) + ro);
        } else {
            const uint2 t = *reinterpret_cast<const uint2 *>(static_cast<const h16 *>(a.R) + ro);
            x.res[0] = t.x;
            x.res[1] = t.y;
        }
        return x;
    };
    Added early{};
    if (NC == 1) early = fetch_added(threadIdx.x);
    auto load_w = [&](int kt) {
#pragma unroll
        for (int j = 0; j < LW; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (lds_void *)(mine + BM * 128 + j * 1024), 16, woff[j], kt * (TBK * 2), 0, 0);
    };
    auto multiply = [&](int kt) {
        const int steps = min(4, (K - kt * TBK) / 16);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s >= steps) break;                              // uniform; only the K tail
            h16x8 xf[TM], wf[TN];
            const int chunk = s * 2 + lhi;
#pragma unroll
            for (int t = 0; t < TM; ++t) xf[t] = *reinterpret_cast<const h16x8 *>(mine + lay(t * 32 + l32, chunk) * 2);
#pragma unroll
            for (int t = 0; t < TN; ++t) wf[t] = *reinterpret_cast<const h16x8 *>(mine + BM * 128 + lay(t * 32 + l32, chunk) * 2);
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j) acc[i][j] = SF_MFMA16(wf[i], xf[j], acc[i][j], 0, 0, 0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // this wave's fragments are in registers: reuse the region
    };
    if constexpr (LN == 0) {
        for (int kt = wave; kt < nkt; kt += NWK) {
#pragma unroll
            for (int j = 0; j < LX; ++j)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void *)(mine + j * 1024), 16, xoff[j], kt * (TBK * 2), 0, 0);
            load_w(kt);
            wait_vmcnt<0>();
            multiply(kt);
        }
    } else {
        // rows of a lane: chunk lane % 8 (8 columns) of rows lane / 8 + 8 i
        constexpr int KPW = 2, RPL = BM / 8;
        const int ch = lane & 7, r8 = lane >> 3;
        const int64_t row0 = (int64_t)tl.b * a.L + tl.m0;
        float2 *stat = reinterpret_cast<float2 *>(smem + (BUF > BM * BN * 4 ? BUF : BM * BN * 4) * NWK);      // [K tile][row] mean and squared deviations of 64 columns
        float xv[KPW][RPL][8];
        h16x8 gv[KPW], bv[KPW];
        if (wave < nkt) load_w(wave);
#pragma unroll
        for (int p = 0; p < KPW; ++p) {
            const int kt = wave + p * NWK, col = kt * TBK + ch * 8;
            if (kt >= nkt) break;                                         // uniform
            gv[p] = *reinterpret_cast<const h16x8 *>(static_cast<const h16 *>(a.ln_g) + col);
            bv[p] = *reinterpret_cast<const h16x8 *>(static_cast<const h16 *>(a.ln_b) + col);
#pragma unroll
            for (int i = 0; i < RPL; ++i) {
                const int64_t at = (row0 + min(r8 + i * 8, a.L - tl.m0 - 1)) * a.lda + col;      // rows beyond the edge: never stored
                if (LN == 1) {
                    const float *x = static_cast<const float *>(a.A) + at;
                    const f32x4 v0 = *reinterpret_cast<const f32x4 *>(x), v1 = *reinterpret_cast<const f32x4 *>(x + 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) { xv[p][i][e] = v0[e]; xv[p][i][4 + e] = v1[e]; }
                } else {
                    const h16x8 v = *reinterpret_cast<const h16x8 *>(static_cast<const h16 *>(a.A) + at);
#pragma unroll
                    for (int e = 0; e < 8; ++e) xv[p][i][e] = (float)v[e];
                }
            }
        }
#pragma unroll
        for (int p = 0; p < KPW; ++p) {
            if (wave + p * NWK >= nkt) break;
#pragma unroll
            for (int i = 0; i < RPL; ++i) {
                float s = 0.f, q = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) s += xv[p][i][e];
                const float m = sum8(s) * (1.0f / TBK);
#pragma unroll
                for (int e = 0; e < 8; ++e) { const float t = xv[p][i][e] - m; q += t * t; }
                q = sum8(q);
                if (ch == 0) stat[(wave + p * NWK) * BM + r8 + i * 8] = make_float2(m, q);
            }
        }
        lds_barrier();
        float mean[RPL], inv[RPL];
#pragma unroll
        for (int i = 0; i < RPL; ++i) {                                   // lane ch joins the K tiles ch and ch + 8
            const float2 t0 = ch < nkt ? stat[ch * BM + r8 + i * 8] : make_float2(0.f, 0.f);
            const float2 t1 = ch + 8 < nkt ? stat[(ch + 8) * BM + r8 + i * 8] : make_float2(0.f, 0.f);
            mean[i] = sum8(t0.x + t1.x) / (float)nkt;
            const float d0 = ch < nkt ? t0.x - mean[i] : 0.f, d1 = ch + 8 < nkt ? t1.x - mean[i] : 0.f;
            const float var = sum8(t0.y + t1.y + (float)TBK * (d0 * d0 + d1 * d1)) / (float)K;
            inv[i] = 1.0f / sqrtf(var + a.ln_eps);
        }
#pragma unroll
        for (int p = 0; p < KPW; ++p) {
            const int kt = wave + p * NWK;
            if (kt >= nkt) break;
            if (p) load_w(kt);
#pragma unroll
            for (int i = 0; i < RPL; ++i) {
                h16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (h16)((xv[p][i][e] - mean[i]) * inv[i] * (float)gv[p][e] + (float)bv[p][e]);
                *reinterpret_cast<h16x8 *>(mine + lay(r8 + i * 8, ch) * 2) = o;
            }
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            multiply(kt);
        }
    }
    barrier();
    // partial tiles: part[wave][token][feature], fp32, 16-byte chunks of a row XOR-ed by the row
    float *part = reinterpret_cast<float *>(smem);
    auto po = [](int row, int c) { return row * BN + ((c ^ (row & (CPR - 1))) << 2); };
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = acc[i][j][q * 4 + e];
                *reinterpret_cast<f32x4 *>(part + wave * BM * BN + po(j * 32 + l32, i * 8 + q * 2 + lhi)) = o;
            }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier();
    if (!tl.vt) {
#pragma unroll 2
        for (int c = threadIdx.x; c < BM * CPR; c += NT) {      // 4 features of a token per thread
            const Added x = NC == 1 ? early : fetch_added(c);
            const int r = c / CPR, cc = c % CPR, i = tl.m0 + r, n = tl.nt0 + cc * 4;
            if (i >= a.L || n >= N) continue;
            const int64_t row = (int64_t)tl.b * a.L + i;
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (float)x.bias[e];
#pragma unroll
            for (int k = 0; k < NWK; ++k) {
                const f32x4 t = *reinterpret_cast<const f32x4 *>(part + k * BM * BN + po(r, cc));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += t[e];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = activate<ACT>(v[e]);
            if (a.R) {
                const h16x4 t16 = __builtin_bit_cast(h16x4, make_uint2(x.res[0], x.res[1]));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += a.r_f32 ? __uint_as_float(x.res[e]) : (float)t16[e];
            }
            const int64_t co = row * a.ldc + a.c0 + n;
            if (a.c_f32) {
                *reinterpret_cast<f32x4 *>(static_cast<float *>(a.C) + co) = v;
            } else {
                h16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (h16)v[e];
                *reinterpret_cast<h16x4 *>(static_cast<h16 *>(a.C) + co) = o;
            }
        }
    } else {
        h16 *V = static_cast<h16 *>(a.VT) + (int64_t)tl.b * a.vt_b;
        for (int c = threadIdx.x; c < BN * (BM / 4); c += NT) {  // one feature of 4 tokens per thread
            const int f = c / (BM / 4), r0 = (c % (BM / 4)) * 4, n = tl.nt0 + f, i = tl.m0 + r0;
            if (n >= N) continue;
            h16 *dst = V + (int64_t)(n - a.vt_from) * a.vt_n + i;
            const float bv = bias ? (float)bias[n] : 0.f;
            h16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = bv;
#pragma unroll
                for (int k = 0; k < NWK; ++k) v += part[k * BM * BN + po(r0 + e, f >> 2) + (f & 3)];
                o[e] = (h16)activate<ACT>(v);
            }
            if (i + 3 < a.L) {
                *reinterpret_cast<h16x4 *>(dst) = o;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < a.L) dst[e] = o[e];
            }
        }
    }
#endif
}

typedef void (*Kernel)(GemmArgs, int, int, int, int);

// `attr_set` belongs to the kernel; setting the attribute twice is harmless
int32_t launch(Kernel kern, std::atomic<bool> &attr_set, const GemmArgs &a, int bm, int bn, int threads, size_t lds, hipStream_t st)
{
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
            hipSuccess)
            return fail(SF_ERR_HIP, "gemm: cannot reserve %zu bytes of LDS", lds);
        attr_set = true;
    }
    const int tiles_m = ceil_div(a.L, bm);
    const int tiles_n = a.VT ? ceil_div(a.vt_from, bn) + ceil_div(a.N - a.vt_from, bn) : ceil_div(a.N, bn);
    const int total = a.B * tiles_m * tiles_n;
    const int per_xcd = a.xcd_rows ? ceil_div(a.B * tiles_m, N_XCD) * tiles_n : ceil_div(total, N_XCD);
    ProfScope prof(SF_KERNEL_GEMM, st);
    hipLaunchKernelGGL(kern, dim3(per_xcd * N_XCD), dim3(threads), lds, st, a, tiles_m, tiles_n, total, per_xcd);
    return SF_OK;
}

template <int ACT>
int32_t launch_pipe(const GemmArgs &a, hipStream_t st)
{
    static std::atomic<bool> set{false};
    return launch(gemm_pipe_kernel<ACT>, set, a, 128, 128, 256, 2 * 256 * TBK * 2, st);
}

template <int TM, int TN, int NWK, int ACT, int LN = 0>
int32_t launch_slice(const GemmArgs &a, hipStream_t st)
{
    static std::atomic<bool> set{false};
    constexpr size_t loads = (size_t)NWK * (TM + TN) * 32 * TBK * 2, parts = (size_t)NWK * TM * TN * 1024 * 4;
    constexpr size_t stats = LN ? (size_t)2 * NWK * TM * 32 * sizeof(float2) : 0;
    return launch(gemm_slice_kernel<TM, TN, NWK, ACT, LN>, set, a, TM * 32, TN * 32, 64 * NWK, (loads > parts ? loads : parts) + stats, st);
}

template <int ACT>
int32_t launch_kind(GemmKind kind, const GemmArgs &a, hipStream_t st)
{
    if (a.ln_g) return a.ln_x32 ? launch_slice<1, 2, 8, ACT, 1>(a, st) : launch_slice<1, 2, 8, ACT, 2>(a, st);
    switch (kind) {
    case GEMM_SLICE8: return launch_slice<1, 2, 8, ACT>(a, st);
    case GEMM_SLICE4: return launch_slice<2, 2, 4, ACT>(a, st);
    default: return launch_pipe<ACT>(a, st);
    }
}

}  // namespace

// 16-byte rows and columns, K a multiple of 32 (the K tail is half a tile), offsets within a tile below 4 GiB
bool gemm_bf16_tile_eligible(const GemmArgs &a)
{
    if (a.epi != EPI_ROWMAJOR || a.K % 32 || a.K < TBK || a.N % 8 || a.n0 % 8 || a.lda % 8 || a.ldw % 8 || a.ldc % 8 || a.c0 % 8 ||
        (a.R && (a.ldr % 8 || a.r0 % 8)))
        return false;
    if (a.VT && (a.R || a.c_f32 || ((a.vt_b | a.vt_n) & 7))) return false;
    if (((uintptr_t)a.A | (uintptr_t)a.W) & 15) return false;              // loads straight into LDS: whole aligned chunks
    // 32-bit byte offsets: within a tile, or (row_map) anywhere in A, which the caller keeps below 4 GiB
    return a.lda < ((int64_t)1 << 23) && a.ldw < ((int64_t)1 << 23);
}

// The LayerNorm rides along where the K tiles of the rows fit the registers of eight waves and there is at most a tile of
// 32 x 64 per compute unit: FFNs of 32 to 2000 rows, d 128 to 1024, then take 0.84 to 0.97 of their time with the launch (d 128
// 11.6 -> 9.9 us, d 512 12.7 -> 11.9), 1.03 to 1.20 from the 257th tile on; tiles of 64 x 64 gain nothing (0.93 to 1.04).
bool gemm_bf16_tile_takes_ln(const GemmArgs &a)
{
    if (a.K % TBK || a.K > 16 * TBK || a.row_map || a.n_lim || a.k_lim || (((uintptr_t)a.ln_g | (uintptr_t)a.ln_b) & 15)) return false;
    const int64_t cols = a.VT ? ceil_div(a.vt_from, 64) + ceil_div(a.N - a.vt_from, 64) : ceil_div(a.N, 64);
    return (int64_t)a.B * ceil_div(a.L, 32) * cols <= 256;
}

int32_t gemm_bf16_tile(GemmKind kind, const GemmArgs &a, hipStream_t st)
{
    switch (a.act) {
    case ACT_RELU: return launch_kind<ACT_RELU>(kind, a, st);
    case ACT_GELU: return launch_kind<ACT_GELU>(kind, a, st);
    default: return launch_kind<ACT_NONE>(kind, a, st);
    }
}

// Which kernel takes a problem: an estimate of each one's time in microseconds, on a whole card of 256 compute units.
// The constants are a fit to 456 launches of layers drawn at random (10 to 130 000 rows, d 128 to 1024, K 128 to 4096, kept heads and channels at
// random), with weights that no cache holds: fixed cost, cost of a K tile and cost of an epilogue per workgroup and
// round.
//   256 x 256: whole rounds of one workgroup per compute unit, 1.06 us per K tile (1.12 with a residual or fp32 output)
//     and 4.9 us per output tile (13.7 with GELU), and the time of the output's own traffic;
//   128 x 128: a chain of 0.57 us per K tile while there is at most one workgroup per compute unit, 0.47 us per K tile
//     and 2.1 us per tile and compute unit beyond (0.59 and 2.5, and a sixth of the output's traffic, with a residual or
//     fp32 output), a last uneven round counted nearly as a whole one;
//   slices: rounds of 256 workgroups (eight slices), dearer from the second on, where the L2 feeds every compute unit
//     with a tile of few rows; or one round of up to two per compute unit (four slices).
// Over those launches the choice costs 0.4 % over the fastest kernel, 16 % at worst, where the gaps between the kernels
// are factors of 3 to 6.
GemmKind gemm_bf16_choose(const GemmArgs &a, bool ws_ok)
{
    auto tiles = [&](int bm, int bn) {
        const int64_t n = a.VT ? ceil_div(a.vt_from, bn) + ceil_div(a.N - a.vt_from, bn) : ceil_div(a.N, bn);
        return (double)(a.B * (int64_t)ceil_div(a.L, bm) * n);
    };
    const bool wide = a.R || a.c_f32;
    const double nk = (a.K + TBK - 1) / TBK, rows = (double)a.B * a.L;
    const bool gelu = a.act == ACT_GELU;
    // reads and writes of the epilogue at the rate of a large copy; those of A and W hide behind the matrix cores
    const double out = rows * a.N * ((a.c_f32 ? 4.0 : 2.0) + (!a.R ? 0.0 : a.r_f32 ? 4.0 : 2.0)) / 5.2e6;
    const double rounds = ceil(tiles(256, 256) / 256);
    const double bare = wide ? 0.93 : 0.73 + 0.27 / (rounds * rounds);
    const double ws = 2.3 + rounds * ((wide ? 1.12 : 1.06) * nk + (gelu ? 13.7 : 4.9)) + bare * out;
    // two workgroups share a compute unit: a last one left alone takes nearly the time of a pair
    double q = tiles(128, 128) / 256;
    if (q > 1) q += 0.87 * (ceil(q) - q) / q;
    const double pipe = 3.8 + (wide ? 0.18 * out : 0.0) +
                        std::max(0.57 * nk + (wide ? 2.5 : gelu ? 2.8 : 1.0), q * (wide ? 0.59 * nk + 2.5 : 0.47 * nk + (gelu ? 3.2 : 2.1)));
    const double r8 = ceil(tiles(32, 64) / 256), c8 = ceil(nk / 8);
    const double s8 = 2.3 + r8 * (r8 > 1 ? 1.9 + 1.35 * c8 : 1.5 + 0.95 * c8);
    const double s4 = (wide ? 3.6 : 4.4) + std::max(1.0, tiles(64, 64) / 256) * (1.7 + 0.98 * ceil(nk / 4));
    GemmKind best = GEMM_PIPE;
    double t = pipe;
    if (ws_ok && ws < t) { best = GEMM_WS; t = ws; }
    if (s4 < t) { best = GEMM_SLICE4; t = s4; }
    if (s8 < t) best = GEMM_SLICE8;
    return best;
}

}  // namespace sf
