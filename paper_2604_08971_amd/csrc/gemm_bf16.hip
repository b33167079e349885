// bf16 MFMA GEMM (fp32 accumulate) for the Q/K/V, output and FFN projections
// of the pruned encoder layer (Sec. 4.4 projections, Sec. 4.5 compacted
// weights).  Both operands are K-contiguous (token-major activations,
// unit-major weights), so every MFMA fragment is one 16-byte LDS read.
//
// Tiling: a workgroup owns a BM x BN output tile of ONE sample (rows never
// straddle samples, because the weight set depends on the sample's presence
// pattern); K is walked in steps of 64 through double-buffered, XOR-swizzled
// LDS tiles; each 64-lane wave owns a (BM/WAVES_M) x (BN/WAVES_N) sub-tile
// as 32x32x16 MFMA blocks.
//
// Orientation: with SWAP = false the MFMA "A" operand is the weight tile, so
// an accumulator lane holds one token and 4 consecutive features: row-major
// stores are 8-byte vectors.  With SWAP = true the roles flip and a lane holds
// one feature and 4 consecutive tokens: that is the store pattern of the
// transposed V layout the attention kernels read.
#include <algorithm>
#include <atomic>

#include "gemm.hpp"

namespace sf {

constexpr int BK = 64;                 // bf16 elements per K step (128 bytes = 8 chunks of 16 B)

__device__ __forceinline__ int swz(int row, int chunk) { return row * BK + ((chunk ^ (row & 7)) << 3); }

__device__ __forceinline__ float apply_act(float z, int act)
{
    if (act == ACT_RELU) return z > 0.f ? z : 0.f;
    if (act == ACT_GELU) return gelu_erf(z);
    return z;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool SWAP>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_bf16_kernel(GemmArgs a)
{
    constexpr int NT = 64 * WAVES_M * WAVES_N;
    constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    constexpr int XCH = BM * 8 / NT, WCH = BN * 8 / NT;      // 16-byte chunks per thread per tile
    static_assert(BM * 8 % NT == 0 && BN * 8 % NT == 0, "tile/threads mismatch");

    extern __shared__ __attribute__((aligned(16))) char smem_raw[];
    h16 *Xs = reinterpret_cast<h16 *>(smem_raw);             // [2][BM*BK]
    h16 *Ws = Xs + 2 * BM * BK;                                 // [2][BN*BK]

    const int tiles_m = (a.L + BM - 1) / BM;
    const int b = blockIdx.x / tiles_m;
    const int m0 = (blockIdx.x % tiles_m) * BM;
    const int nt0 = blockIdx.y * BN;                               // first feature of this tile (within launch)
    const int p = a.pattern_id ? a.pattern_id[b] : 0;
    if (p < 0) return;                                             // sample not in use
    if (a.n_lim) a.N = min(a.N, a.n_lim[p]);
    if (a.k_lim) a.K = min(a.K, a.k_lim[p]);
    if (nt0 >= a.N) return;

    const h16 *A = static_cast<const h16 *>(a.A) + ((int64_t)b * a.L) * a.lda;
    const h16 *W = static_cast<const h16 *>(a.W) + (int64_t)p * a.w_pstride + (int64_t)a.n0 * a.ldw;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int l32 = lane & 31, lhi = lane >> 5;

    uint4 xr[XCH], wr[WCH];
    const int lc = tid & 7;                 // chunk within the 128-byte row
    const int lr = tid >> 3;                // first row handled by this thread

    auto load_global = [&](int k0) {
        const int k = k0 + lc * 8;
        const bool kin = k < a.K;
#pragma unroll
        for (int j = 0; j < XCH; ++j) {
            const int r = lr + j * (NT / 8);
            const int i = m0 + r;
            xr[j] = (kin && i < a.L) ? *reinterpret_cast<const uint4 *>(A + (int64_t)i * a.lda + k)
                                     : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < WCH; ++j) {
            const int r = lr + j * (NT / 8);
            const int n = nt0 + r;
            wr[j] = (kin && n < a.N) ? *reinterpret_cast<const uint4 *>(W + (int64_t)n * a.ldw + k)
                                     : make_uint4(0, 0, 0, 0);
        }
    };
    auto store_lds = [&](int buf) {
        h16 *xs = Xs + buf * BM * BK, *ws = Ws + buf * BN * BK;
#pragma unroll
        for (int j = 0; j < XCH; ++j) {
            const int r = lr + j * (NT / 8);
            *reinterpret_cast<uint4 *>(xs + swz(r, lc)) = xr[j];
        }
#pragma unroll
        for (int j = 0; j < WCH; ++j) {
            const int r = lr + j * (NT / 8);
            *reinterpret_cast<uint4 *>(ws + swz(r, lc)) = wr[j];
        }
    };

    // accumulators: [row-operand tile][col-operand tile]
    constexpr int TP = SWAP ? TM : TN, TQ = SWAP ? TN : TM;
    f32x16 acc[TP][TQ];
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TQ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int nk = (a.K + BK - 1) / BK;
    load_global(0);
    store_lds(0);
    __syncthreads();

    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) load_global((kt + 1) * BK);
        const h16 *xs = Xs + (kt & 1) * BM * BK, *ws = Ws + (kt & 1) * BN * BK;
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            h16x8 xf[TM], wf[TN];
            const int chunk = s * 2 + lhi;
#pragma unroll
            for (int t = 0; t < TM; ++t)
                xf[t] = *reinterpret_cast<const h16x8 *>(xs + swz(wm * WTM + t * 32 + l32, chunk));
#pragma unroll
            for (int t = 0; t < TN; ++t)
                wf[t] = *reinterpret_cast<const h16x8 *>(ws + swz(wn * WTN + t * 32 + l32, chunk));
#pragma unroll
            for (int i = 0; i < TP; ++i)
#pragma unroll
                for (int j = 0; j < TQ; ++j) {
                    if (SWAP) acc[i][j] = SF_MFMA16(xf[i], wf[j], acc[i][j], 0, 0, 0);
                    else      acc[i][j] = SF_MFMA16(wf[i], xf[j], acc[i][j], 0, 0, 0);
                }
        }
        if (kt + 1 < nk) store_lds((kt + 1) & 1);
        __syncthreads();
    }

    // ---- epilogue -------------------------------------------------------------
    const h16 *bias = a.bias ? static_cast<const h16 *>(a.bias) + (int64_t)p * a.bias_pstride + a.n0 : nullptr;
    if (!SWAP) {
        // lane: token i = m0 + wm*WTM + tm*32 + l32 ; features n = wn*WTN + tn*32 + q*8 + lhi*4 + {0..3}
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int i = m0 + wm * WTM + tm * 32 + l32;
            if (i >= a.L) continue;
            const int64_t row = (int64_t)b * a.L + i;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = nt0 + wn * WTN + tn * 32 + q * 8 + lhi * 4;
                    if (n >= a.N) continue;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[tn][tm][q * 4 + e];
                    if (bias) {
                        const h16x4 bv = *reinterpret_cast<const h16x4 *>(bias + n);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += (float)bv[e];
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = apply_act(v[e], a.act);
                    if (a.R) {
                        const int64_t ro = row * a.ldr + a.r0 + n;
                        if (a.r_f32) {
                            const f32x4 rv = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.R) + ro);
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] += rv[e];
                        } else {
                            const h16x4 rv = *reinterpret_cast<const h16x4 *>(static_cast<const h16 *>(a.R) + ro);
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] += (float)rv[e];
                        }
                    }
                    const int64_t co = row * a.ldc + a.c0 + n;
                    if (a.c_f32) {
                        f32x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = v[e];
                        *reinterpret_cast<f32x4 *>(static_cast<float *>(a.C) + co) = o;
                    } else {
                        h16x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = (h16)v[e];
                        *reinterpret_cast<h16x4 *>(static_cast<h16 *>(a.C) + co) = o;
                    }
                }
            }
        }
    } else {
        // lane: feature n = wn*WTN + tn*32 + l32 ; tokens i = m0 + wm*WTM + tm*32 + q*8 + lhi*4 + {0..3}
        h16 *C = static_cast<h16 *>(a.C) + (int64_t)b * a.vt_b;
        const bool vec_ok = ((a.vt_b | a.vt_n) & 3) == 0;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int n = nt0 + wn * WTN + tn * 32 + l32;
            if (n >= a.N) continue;
            const float bv = bias ? (float)bias[n] : 0.f;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = m0 + wm * WTM + tm * 32 + q * 8 + lhi * 4;
                    if (i >= a.L) continue;
                    h16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = (h16)apply_act(acc[tm][tn][q * 4 + e] + bv, a.act);
                    h16 *dst = C + (int64_t)n * a.vt_n + i;
                    if (vec_ok && i + 3 < a.L) {
                        *reinterpret_cast<h16x4 *>(dst) = o;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (i + e < a.L) dst[e] = o[e];
                    }
                }
            }
        }
    }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool SWAP>
static int32_t launch_cfg(const GemmArgs &a, hipStream_t st)
{
    auto kern = gemm_bf16_kernel<BM, BN, WAVES_M, WAVES_N, SWAP>;
    constexpr size_t lds = (size_t)2 * (BM + BN) * BK * sizeof(h16);
    static std::atomic<bool> attr_set{false};     // per template instance; setting the attribute twice is harmless
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return fail(SF_ERR_HIP, "gemm: cannot reserve %zu bytes of LDS", lds);
        attr_set = true;
    }
    dim3 grid(ceil_div(a.L, BM) * a.B, ceil_div(a.N, BN));
    ProfScope prof(SF_KERNEL_GEMM, st);
    hipLaunchKernelGGL(kern, grid, dim3(64 * WAVES_M * WAVES_N), lds, st, a);
    return SF_OK;
}

bool gemm_takes_row_map(int dtype, const GemmArgs &a)
{
    return dtype == SF_BF16 && a.epi == EPI_ROWMAJOR && a.a_rows > 0 && (gemm_bf16_ws_eligible(a) || gemm_bf16_tile_eligible(a));
}
bool gemm_takes_vt_split(int dtype, const GemmArgs &a)
{
    return dtype == SF_BF16 && a.epi == EPI_ROWMAJOR && (gemm_bf16_ws_eligible(a) || gemm_bf16_tile_eligible(a)) &&
           a.vt_from > 0 && a.vt_from < a.N && a.vt_from % 8 == 0 && a.vt_b % 8 == 0 && a.vt_n % 8 == 0 && !a.R &&
           !a.c_f32 && !a.n_lim;
}

// One weight set and row-major output: the samples are one long one, and no tile is cut at a sample's end
static void join_samples(GemmArgs &a)
{
    if (!a.pattern_id && a.epi == EPI_ROWMAJOR && !a.VT && !a.row_map && (int64_t)a.B * a.L * a.lda * 2 < ((int64_t)1 << 32)) {
        a.L *= a.B;
        a.B = 1;
    }
}

// The kernel of a problem, which may become one long sample
static GemmKind choose(GemmArgs &a)
{
    join_samples(a);
    const bool ws_ok = gemm_bf16_ws_eligible(a);
    if (gemm_bf16_tile_eligible(a)) return gemm_bf16_choose(a, ws_ok);
    return ws_ok ? GEMM_WS : GEMM_GENERIC;
}

bool gemm_takes_ln(int dtype, const GemmArgs &a0)
{
    GemmArgs a = a0;
    if (dtype == SF_F32) return gemm_f32_takes_ln(a);
    if (dtype != SF_BF16 || a.epi != EPI_ROWMAJOR || (a.VT && !gemm_takes_vt_split(dtype, a))) return false;
    join_samples(a);
    return gemm_bf16_tile_eligible(a) && gemm_bf16_tile_takes_ln(a);
}

// Row tiles of gemm_bf16_rows.hip: 64 rows and two workgroups per compute unit up to N 256, 128 rows and one beyond, where a last
// round that is not full costs nearly a whole one.
static int64_t row_tiles(const GemmArgs &a) { return a.B * (int64_t)ceil_div(a.L, a.N <= 256 ? 64 : 128); }
// Share of their rows that are there: short samples with weights of their own leave most of a tile empty
static double tile_fill(const GemmArgs &a) { return (double)a.B * a.L / (row_tiles(a) * (a.N <= 256 ? 64. : 128.)); }
static bool rounds_filled(int64_t tiles, double share) { return tiles >= share * 256 * ((tiles + 255) / 256); }
// Whole rows give the bits of the kernel that gemm() takes for the product on its own: beyond N 256 there are no registers for a sum per K
// slice (a batch of many short samples, whose 128-row tiles are mostly empty, would be sliced).
static bool rows_keep_bits(const GemmArgs &a0, int64_t N)
{
    GemmArgs a = a0;
    const GemmKind kind = choose(a);
    return kind == GEMM_WS || kind == GEMM_PIPE || (N <= 256 && kind != GEMM_GENERIC);
}

// The product with the LayerNorm of its rows against the two launches, us: 12 288 rows, N 128, K 64 6.2 / 12.1; 24 576 rows in samples of 384,
// N 256, K 192 17.3 / 22; 65 536 rows, N 512, K 384 86 / 111; 122 880 in samples of 480, K 256 138 / 193.  Beyond N 256 by how full
// the rounds are, one line for both widths, where the slower of them is ahead in one round and even in two.  This / two launches, rounds
// filled 0.63 0.69 0.75 0.81 0.91 1.0 (one) and 0.55 0.63 0.72 0.78 0.86 1.0 (two):
//   N 384, K 192   1.07 0.87 0.86 0.85 0.85 0.86    1.13 1.08 1.00 0.97 0.95 0.92
//   N 512, K 320   0.95 0.94 0.91 0.92 0.91 0.90    1.18 1.11 1.04 0.99 0.87 0.80
// Up to N 256 a few tiles take a few steps only, since a tile walks K alone (N 256, 128 tiles: K 512 0.80, 1024 0.96, 2048 1.25; N 128, 32
// tiles: K 128 0.80, 512 0.97, 1024 1.18; with the sums of K slices 34 samples of 53 rows, four layers, 205 us with K 640 so, 192
// without), and below 32 tiles the LayerNorm rides along with the product that follows, which costs less than this kernel's epilogue.
// An empty row costs a tile here what a full one does, the smaller tiles and K slices of gemm() less.  A layer without / with this, us:
// 253 samples of 18 rows, d 512, K 768 117 / 132; 227 of 67 rows, d 384, K 128 73 / 80; 160 of 12 rows, d 256, K 192 39.6 / 40.9.  Of 408
// layers drawn at random (samples of 8 to 700 rows) 34 took over 2 % longer, the worst 1.13, and of the 336 that a bound on the empty rows
// leaves 5, the worst 1.03.
bool gemm_takes_ln_out(int dtype, const GemmArgs &a0)
{
    GemmArgs a = a0;
    if (dtype != SF_BF16 || !gemm_bf16_rows_eligible(a)) return false;
    join_samples(a);
    const int64_t tiles = row_tiles(a);
    if (tile_fill(a) < (a.N <= 256 ? 0.25 : 0.75)) return false;
    if (a.N <= 256 ? tiles < 32 || a.K > (a.N == 128 ? 4 : 2) * tiles + 64 : !rounds_filled(tiles, 0.77)) return false;
    return rows_keep_bits(a0, a.N);
}

// Both products see the samples joined where the up-projection does
static void join_ffn(GemmArgs &up, GemmArgs &down)
{
    join_samples(up);
    down.B = up.B;
    down.L = up.L;
}

// The FFN in one launch against two (and a LayerNorm of its rows), us: 24 576 rows in samples of 384, d 256, 640 channels 34 / 37 (37 / 47);
// 65 536 rows, d 256, 640 channels 72 / 90 (78 / 115); 65 536 rows, d 512, 1280 channels 196 / 208 (208 / 238); 122 880 in
// samples of 480, 1024 channels 317 / 345 (338 / 408).  A tile walks its hidden channels alone, 1.9 us per 128 of them at d 128 and
// 3.3 at d 256 however few tiles there are, where the two launches spread them over columns and K slices: few tiles take few channels.
// One launch / two, with the LayerNorm:
//   d 128   channels   256  512  1024  2048  4096        d 256   channels   512  1024  2048  4096  8192
//    32 tiles         0.77 1.04  1.52  2.27  2.87        128 tiles         0.95  1.12  1.17  1.74  1.89
//    64               0.72 0.99  1.39  1.81  1.88        160               0.82  0.86  0.99  1.19  1.20
//    96               0.63 0.81  1.05  1.22  1.51        192               0.75  0.87  0.93  1.15  1.14
//   128               0.61 0.77  0.97  0.96  1.17        256               0.74  0.73  0.84  1.08  1.03
//   192               0.56 0.66  0.74  0.87  0.88        320               0.77  0.93  0.84  0.95  0.94
// (ReLU, full tiles; without the LayerNorm 0.05 to 0.15 more below 192 tiles).  GELU stands between the two products here and costs as much
// as a third more channels; a tile with empty rows costs what a full one does, where the separate launches have smaller tiles: both are
// counted as channels.  us, two launches / one: 247 samples of 24 rows, d 512, 3776 channels, GELU 90 / 244; 227 of 9 rows, d 128, 2048 channels 16 / 49;
// 189 of 31, d 256, 1408 channels 28 / 45.  At d 256 a few compute units with two tiles, and a few with two more, cost as much as all:
// 60 samples of 646 rows (660 tiles), 3904 channels 292 / 325; 33 072 rows (517 tiles), 2112 channels 150 / 169; 91 samples of 195 rows (364), 896
// channels 50 / 57 (all GELU).  Of 1169 calls and layers
// drawn at random (samples of 8 to 700 rows, 64 to 4096 channels) 165 took over 2 % longer by the tiles alone, the worst 3.1 times as long; of the
// 813 that these bounds leave 12, the worst 1.06.
// Beyond d 256 by how full the rounds are, with one line for both widths, which leaves the narrower one some of its gain.  With the
// LayerNorm, rounds filled as above:
//   d 384,  960 channels   0.96 0.78 0.70 0.71 0.71 0.69    0.98 0.89 0.84 0.77 0.76 0.71
//   d 512, 1280 channels   0.90 0.91 0.87 0.82 0.80 0.79    1.08 0.97 0.97 0.95 0.87 0.87
// and without it 1.03 0.81 0.73 0.74 0.74 0.73, 1.04 0.95 0.90 0.83 0.81 0.76 and 0.94 0.97 0.93 0.87 0.84 0.85, 1.14 1.02 1.04 1.01 0.93 0.95.
bool ffn_in_one(int dtype, const GemmArgs &up0, const GemmArgs &down0)
{
    GemmArgs up = up0, down = down0;
    if (dtype != SF_BF16 || !ffn_bf16_rows_eligible(up, down)) return false;
    join_ffn(up, down);
    const int64_t tiles = row_tiles(down);
    const bool ln = down.lno_y, gelu = up.act == ACT_GELU;
    const double fill = tile_fill(down), F = up.N * (gelu ? 4. / 3 : 1.) / fill;
    if (fill < (down.N <= 256 ? 1. / 3 : 0.5)) return false;
    if (down.N == 128) {
        if (tiles < 32 || F > (tiles > 256 ? 4096 : tiles >= 192 ? 2048 : ln ? 6 * tiles + 192 : 5 * tiles + 96)) return false;
    } else if (down.N == 256) {
        const int64_t one_round = std::min<int64_t>(2048, ln ? 20 * (tiles - 104) : 32 * (tiles - 116));
        const int64_t more = tiles < (gelu ? 400 : 340) ? 1365 : tiles > 512 && tiles <= 640 ? 1792 : 2816;
        if (tiles < 128 || F > (tiles > 256 ? more : one_round)) return false;
    } else if (!rounds_filled(tiles, ln ? 0.8 : 0.93) || F / fill > 3840 || (fill < 0.6 && F > 1536)) {
        return false;
    }
    return rows_keep_bits(up, down.N) && rows_keep_bits(down, down.N);
}

int32_t ffn_one_launch(const GemmArgs &up0, const GemmArgs &down0, hipStream_t st)
{
    GemmArgs up = up0, down = down0;
    join_ffn(up, down);
    GemmArgs u = up, d = down;
    return ffn_bf16_rows(up, choose(u), down, choose(d), st);
}

int32_t gemm_bf16(const GemmArgs &a0, hipStream_t st)
{
    GemmArgs a = a0;
    if (a.B <= 0 || a.N <= 0) return SF_OK;
    if (a.VT && !gemm_takes_vt_split(SF_BF16, a)) return fail(SF_ERR_UNSUPPORTED, "gemm(bf16): transposed column range on a problem the tiled kernels do not take");
    if (a.row_map && !gemm_takes_row_map(SF_BF16, a)) return fail(SF_ERR_UNSUPPORTED, "gemm(bf16): row_map on a problem the tiled kernels do not take");
    if (a.ln_g) {
        if (!gemm_takes_ln(SF_BF16, a)) return fail(SF_ERR_UNSUPPORTED, "gemm(bf16): LayerNorm on a problem that does not take it along");
        join_samples(a);
        return gemm_bf16_tile(GEMM_SLICE8, a, st);
    }
    if (a.lno_y) {
        if (!gemm_takes_ln_out(SF_BF16, a)) return fail(SF_ERR_UNSUPPORTED, "gemm(bf16): LayerNorm of the output on a problem that does not write it");
        const GemmKind kind = choose(a);
        return gemm_bf16_rows(a, kind, st);
    }
    const GemmKind kind = choose(a);
    if (kind == GEMM_WS) return gemm_bf16_ws(a, st);
    if (kind != GEMM_GENERIC) return gemm_bf16_tile(kind, a, st);
    if (a.K % 8 || a.lda % 8 || a.ldw % 8 || a.N % 4 || a.n0 % 4 || (a.R && (a.ldr % 4 || a.r0 % 4)) ||
        (a.epi == EPI_ROWMAJOR && (a.ldc % 4 || a.c0 % 4)))
        return fail(SF_ERR_SHAPE, "gemm(bf16): K, leading dimensions and column origins must be multiples of 8/4");
    const bool swap = a.epi == EPI_VT;
    if (swap && (a.R || a.c_f32)) return fail(SF_ERR_UNSUPPORTED, "gemm(bf16): residual / fp32 output with transposed store");
    return swap ? launch_cfg<128, 128, 2, 2, true>(a, st) : launch_cfg<128, 128, 2, 2, false>(a, st);
}

}  // namespace sf

using namespace sf;

extern "C" int32_t sf_gemm_kernel(const sf_desc *desc, int32_t N, int32_t K, int32_t act, int32_t residual)
{
    Dims D;
    if (int32_t rc = read_desc(desc, D)) return rc;
    if (N < 1 || K < 1) return fail(SF_ERR_INVALID_ARG, "gemm_kernel: N and K must be positive");
    if (D.dtype != SF_BF16) return fail(SF_ERR_UNSUPPORTED, "gemm_kernel: 16-bit models only");
    GemmArgs a{};
    a.B = D.B; a.L = D.L; a.N = N; a.K = K; a.lda = a.ldw = K; a.ldc = a.ldr = N; a.act = act;
    a.R = residual ? &a : nullptr; a.r_f32 = a.c_f32 = residual != 0;               // only looked at, never followed
    a.pattern_id = D.P > 1 ? &D.P : nullptr;
    return choose(a);
}
