// fp32 GEMM (plain FMA, LDS-tiled) and LayerNorm for both dtypes.
// The fp32 path exists for the 1e-5 parity bar of the fp32 workload; it is
// not the throughput path.
#include "gemm.hpp"

namespace sf {

int32_t gemm_bf16(const GemmArgs &a, hipStream_t st);

constexpr int FT = 32;      // output tile edge
constexpr int FK = 64;      // K step

__device__ __forceinline__ float act_f32(float z, int act)
{
    if (act == ACT_RELU) return z > 0.f ? z : 0.f;
    if (act == ACT_GELU) return 0.5f * z * (1.f + erff(z * 0.70710678118654752f));
    return z;
}

// Sum over the eight lanes 8 i .. 8 i + 7, in each of them, joined as by the last steps of wave_sum()
__device__ __forceinline__ float sum8(float x)
{
    x += __shfl_xor(x, 4);
    x += __shfl_xor(x, 2);
    return x + __shfl_xor(x, 1);
}

constexpr int FLN = 256;    // longest row whose LayerNorm the product takes along

// 256 threads; thread (tx,ty) of a 16x16 grid owns rows ty, ty + 16 and columns tx, tx + 16 of the 32x32 tile: any 16 lanes then read
// 16 different 16-byte slots of LDS (rows of 272 bytes).  Small problems are a chain of memory round trips, one per K step: a step
// is 64 of K, all 16 loads of a thread are in flight before the first is used, and those of the next step are issued before this one's
// products.  Four values of K per LDS read; every sum runs over K in order.  2 samples of 48 rows, N 64 to 128, K 32 to 128: 6.1-7.2 us
// with single values, 4.6-7.0 now (the small encoder of those 43.7 -> 37.1 us with the LayerNorms along).
// LN: the rows of A come unnormalised.  Eight threads hold a row (K <= FLN) and take mean and deviations from loads that are in
// flight with the first step's; every column of tiles does so again, which costs less than the launch it replaces (3.2 us) while there
// are few of them.  Thread c of the eight stands for lanes c, c + 8, .. of the launch and adds in its order, so that both give the
// same bits: as layernorm_vec_kernel (LN_VEC: eight columns in a row per lane) or, where rows are no whole chunks of 16 bytes,
// layernorm_kernel (LN_ONE: columns 64 apart).
enum { LN_NONE, LN_VEC, LN_ONE };
template <int LN>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs a)
{
    __shared__ __attribute__((aligned(16))) float Xs[FT][FK + 4], Ws[FT][FK + 4];
    __shared__ float mean[FT], inv[FT];
    const int tiles_m = (a.L + FT - 1) / FT;
    const int b = blockIdx.x / tiles_m;
    const int m0 = (blockIdx.x % tiles_m) * FT;
    const int nt0 = blockIdx.y * FT;
    const int p = a.pattern_id ? a.pattern_id[b] : 0;
    if (p < 0) return;                                             // sample not in use
    if (a.n_lim) a.N = min(a.N, a.n_lim[p]);
    if (a.k_lim) a.K = min(a.K, a.k_lim[p]);
    if (nt0 >= a.N) return;
    const float *A = static_cast<const float *>(a.A) + ((int64_t)b * a.L) * a.lda;
    const float *W = static_cast<const float *>(a.W) + (int64_t)p * a.w_pstride + (int64_t)a.n0 * a.ldw;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    float acc[2][2] = {{0.f, 0.f}, {0.f, 0.f}};

    constexpr int NL = FT * FK / 256;
    float xv[NL], wv[NL], gk = 1.f, bk = 0.f;                      // column k0 + threadIdx.x % FK is the same in all NL loads
    auto fetch = [&](int k0) {
        const int k = k0 + threadIdx.x % FK;
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int r = (threadIdx.x + u * 256) / FK, i = m0 + r, n = nt0 + r;
            xv[u] = (i < a.L && k < a.K) ? A[(int64_t)i * a.lda + k] : 0.f;
            wv[u] = (n < a.N && k < a.K) ? W[(int64_t)n * a.ldw + k] : 0.f;
        }
        if (LN != LN_NONE && k < a.K) {
            gk = static_cast<const float *>(a.ln_g)[k];
            bk = static_cast<const float *>(a.ln_b)[k];
        }
    };
    fetch(0);
    // what the epilogue adds is on its way with the first step: read at the end it is a memory round trip of its own
    const float *bias = a.bias ? static_cast<const float *>(a.bias) + (int64_t)p * a.bias_pstride + a.n0 : nullptr;
    const float *R = static_cast<const float *>(a.R);
    float bv[2], rv[2][2];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int n = nt0 + tx + v * 16;
        bv[v] = bias && n < a.N ? bias[n] : 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = m0 + ty + u * 16;
            rv[u][v] = R && i < a.L && n < a.N ? R[((int64_t)b * a.L + i) * a.ldr + a.r0 + n] : 0.f;
        }
    }
    if constexpr (LN != LN_NONE) {
        constexpr int NP = LN == LN_VEC ? 4 : 8, PL = FLN / 8 / NP;         // lanes of the launch per thread, columns per lane
        const int r = threadIdx.x / 8, c = threadIdx.x % 8;
        const float *x = A + (int64_t)min(m0 + r, a.L - 1) * a.lda;
        auto column = [&](int i, int j) { return LN == LN_VEC ? (c + 8 * i) * 8 + j : c + 8 * i + 64 * j; };
        float v[NP][PL], part[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if constexpr (LN == LN_VEC) {
#pragma unroll
                for (int j = 0; j < PL; j += 4) {
                    f32x4 t = {0.f, 0.f, 0.f, 0.f};
                    if (column(i, 0) < a.K) t = *reinterpret_cast<const f32x4 *>(x + column(i, j));
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[i][j + e] = t[e];
                }
            } else {
#pragma unroll
                for (int j = 0; j < PL; ++j) v[i][j] = column(i, j) < a.K ? x[column(i, j)] : 0.f;
            }
        // lanes 32, 16 and 8 apart are with the same thread (none 32 apart of rows of up to 256 columns by eights)
        auto joined = [&]() {
            if constexpr (LN == LN_VEC) return sum8((part[0] + part[2]) + (part[1] + part[3]));
            else return sum8(((part[0] + part[4]) + (part[2] + part[6])) + ((part[1] + part[5]) + (part[3] + part[7])));
        };
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            part[i] = v[i][0];
#pragma unroll
            for (int j = 1; j < PL; ++j) part[i] += v[i][j];
        }
        const float m = joined() / a.K;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            float t[PL];
#pragma unroll
            for (int j = 0; j < PL; ++j) t[j] = column(i, j) < a.K ? v[i][j] - m : 0.f;
            part[i] = LN == LN_VEC ? squares4(t) : t[0] * t[0];
#pragma unroll
            for (int j = LN == LN_VEC ? 4 : 1; j < PL; ++j) part[i] = __builtin_fmaf(t[j], t[j], part[i]);
        }
        const float q = joined();
        if (c == 0) {
            mean[r] = m;
            inv[r] = 1.0f / sqrtf(q / a.K + a.ln_eps);
        }
        __syncthreads();
    }
    auto operand = [&](float x, int r) {
        if constexpr (LN == LN_NONE) return x;
        const float n = (x - mean[r]) * inv[r];
        if constexpr (LN == LN_VEC) return __builtin_fmaf(n, gk, bk);
        {
#pragma clang fp contract(off)
            const float scaled = n * gk;
            return scaled + bk;
        }
    };
    for (int k0 = 0; k0 < a.K; k0 += FK) {
        const int k = threadIdx.x % FK;
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int r = (threadIdx.x + u * 256) / FK;
            Xs[r][k] = LN == LN_NONE || k0 + k < a.K ? operand(xv[u], r) : 0.f;       // behind K: no multiple of the mean
            Ws[r][k] = wv[u];
        }
        __syncthreads();
        if (k0 + FK < a.K) fetch(k0 + FK);
        for (int kq = 0; kq < min(FK, a.K - k0); kq += 16)       // K of 16 or 40 has no use for the rest of the step
#pragma unroll
            for (int kk = kq; kk < kq + 16; kk += 4) {
                f32x4 x[2], w[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    x[u] = *reinterpret_cast<const f32x4 *>(&Xs[ty + u * 16][kk]);
                    w[u] = *reinterpret_cast<const f32x4 *>(&Ws[tx + u * 16][kk]);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int v = 0; v < 2; ++v) acc[u][v] = fmaf(x[u][e], w[v][e], acc[u][v]);
            }
        __syncthreads();
    }
    float *C = static_cast<float *>(a.C);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int i = m0 + ty + u * 16, n = nt0 + tx + v * 16;
            if (i >= a.L || n >= a.N) continue;
            const int64_t row = (int64_t)b * a.L + i;
            float z = act_f32(acc[u][v] + bv[v], a.act);
            if (R) z += rv[u][v];
            if (a.epi == EPI_VT) C[(int64_t)b * a.vt_b + (int64_t)n * a.vt_n + i] = z;
            else C[row * a.ldc + a.c0 + n] = z;
        }
}

// Few columns of tiles only: each forms the statistics of its rows again
bool gemm_f32_takes_ln(const GemmArgs &a)
{
    return a.K <= FLN && !a.k_lim && !a.n_lim && (int64_t)a.B * ceil_div(a.L, FT) * ceil_div(a.N, FT) <= 1024;
}

int32_t gemm(int dtype, const GemmArgs &a, hipStream_t st)
{
    if (dtype == SF_BF16) return gemm_bf16(a, st);
    if (a.row_map || a.VT) return fail(SF_ERR_UNSUPPORTED, "gemm(f32): row_map / transposed column range are not supported");
    if (a.B <= 0 || a.N <= 0) return SF_OK;
    dim3 grid(ceil_div(a.L, FT) * a.B, ceil_div(a.N, FT));
    if (a.ln_g) {
        if (!gemm_f32_takes_ln(a)) return fail(SF_ERR_UNSUPPORTED, "gemm(f32): LayerNorm on a problem that does not take it along");
        // as launch_ln() chooses; the launch would write rows of its own that are aligned
        const bool vec = a.K % 8 == 0 && a.lda % 4 == 0 && !(((uintptr_t)a.A | (uintptr_t)a.ln_g | (uintptr_t)a.ln_b) & 15);
        if (vec) hipLaunchKernelGGL(gemm_f32_kernel<LN_VEC>, grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL(gemm_f32_kernel<LN_ONE>, grid, dim3(256), 0, st, a);
    } else {
        hipLaunchKernelGGL(gemm_f32_kernel<LN_NONE>, grid, dim3(256), 0, st, a);
    }
    return SF_OK;
}

// One 64-lane wave per row; statistics in fp32; biased variance.
// TI: stored type of x, TP: type of gamma/beta, TO: type of y.  y may alias x
// when TI == TO (each row is read completely before it is written).
template <class TI, class TP, class TO>
__global__ __launch_bounds__(256) void layernorm_kernel(const TI *x, const TP *__restrict__ gamma,
                                                        const TP *__restrict__ beta, float eps, int64_t rows,
                                                        int d, TO *y)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const TI *xr = x + row * d;
    TO *yr = y + row * d;
    float s = 0.f;
    for (int k = lane; k < d; k += 64) s += to_f32(xr[k]);
    s = wave_sum(s);
    const float mean = s / d;
    float v = 0.f;
    for (int k = lane; k < d; k += 64) { const float c = to_f32(xr[k]) - mean; v += c * c; }
    v = wave_sum(v);
    const float inv = 1.0f / sqrtf(v / d + eps);
    for (int k = lane; k < d; k += 64) {
        float z = (to_f32(xr[k]) - mean) * inv;
        if (gamma) z *= to_f32(gamma[k]);
        if (beta) z += to_f32(beta[k]);
        yr[k] = from_f32<TO>(z);
    }
}

// 8 consecutive parameters as floats (`fill` when the vector is absent); 16-byte aligned offsets
template <class TP>
__device__ __forceinline__ void load8(const TP *p, int off, float fill, float (&out)[8])
{
    if (!p) {
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = fill;
    } else if constexpr (sizeof(TP) == 2) {
        const h16x8 t = *reinterpret_cast<const h16x8 *>(p + off);
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = (float)t[e];
    } else {
        const f32x4 t0 = *reinterpret_cast<const f32x4 *>(p + off), t1 = *reinterpret_cast<const f32x4 *>(p + off + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { out[e] = t0[e]; out[4 + e] = t1[e]; }
    }
}

// Vector variant for d % 8 == 0 and d <= 64 * 8 * NCH: the row is read once with
// 16/32-byte loads, kept in registers for both statistics passes, and written
// with 16-byte stores.  One wave per row, 4 rows per block.
template <class TI, class TP, class TO, int NCH>
__global__ __launch_bounds__(256) void layernorm_vec_kernel(const TI *x, const TP *__restrict__ gamma,
                                                            const TP *__restrict__ beta, float eps, int64_t rows,
                                                            int d, TO *y)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const TI *xr = x + row * d;
    TO *yr = y + row * d;
    const int nch = d >> 3;                       // chunks of 8 elements
    float v[NCH][8];
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int ch = lane + c * 64;
        if (ch < nch) {
            if constexpr (sizeof(TI) == 2) {
                const h16x8 t = *reinterpret_cast<const h16x8 *>(xr + ch * 8);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[c][e] = (float)t[e];
            } else {
                const f32x4 t0 = *reinterpret_cast<const f32x4 *>(xr + ch * 8);
                const f32x4 t1 = *reinterpret_cast<const f32x4 *>(xr + ch * 8 + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) { v[c][e] = t0[e]; v[c][4 + e] = t1[e]; }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) s += v[c][e];
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[c][e] = 0.f;
        }
    }
    s = wave_sum(s);
    const float mean = s / d;
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (lane + c * 64 < nch) {
            float t[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] = v[c][e] - mean;
            if (c == 0) q = squares4(t);
#pragma unroll
            for (int e = c == 0 ? 4 : 0; e < 8; ++e) q = __builtin_fmaf(t[e], t[e], q);
        }
    q = wave_sum(q);
    const float inv = 1.0f / sqrtf(q / d + eps);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int ch = lane + c * 64;
        if (ch >= nch) continue;
        float z[8], gm[8], bt[8];
        load8(gamma, ch * 8, 1.f, gm);
        load8(beta, ch * 8, 0.f, bt);
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = (v[c][e] - mean) * inv * gm[e] + bt[e];
        if constexpr (sizeof(TO) == 2) {
            h16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (h16)z[e];
            *reinterpret_cast<h16x8 *>(yr + ch * 8) = o;
        } else {
            f32x4 o0, o1;
#pragma unroll
            for (int e = 0; e < 4; ++e) { o0[e] = z[e]; o1[e] = z[4 + e]; }
            *reinterpret_cast<f32x4 *>(yr + ch * 8) = o0;
            *reinterpret_cast<f32x4 *>(yr + ch * 8 + 4) = o1;
        }
    }
}

template <class TI, class TP, class TO>
static void launch_ln(const void *x, const void *gamma, const void *beta, float eps, int64_t rows, int d, void *y,
                      hipStream_t st)
{
    dim3 grid((unsigned)((rows + 3) / 4));
    const bool vec = d % 8 == 0 && ((uintptr_t)x % 16 == 0) && ((uintptr_t)y % 16 == 0) &&
                     ((uintptr_t)gamma % 16 == 0) && ((uintptr_t)beta % 16 == 0);
#define SF_LN_ARGS grid, dim3(256), 0, st, (const TI *)x, (const TP *)gamma, (const TP *)beta, eps, rows, d, (TO *)y
    if (vec && d <= 512) hipLaunchKernelGGL((layernorm_vec_kernel<TI, TP, TO, 1>), SF_LN_ARGS);
    else if (vec && d <= 1024) hipLaunchKernelGGL((layernorm_vec_kernel<TI, TP, TO, 2>), SF_LN_ARGS);
    else if (vec && d <= 2048) hipLaunchKernelGGL((layernorm_vec_kernel<TI, TP, TO, 4>), SF_LN_ARGS);
    else hipLaunchKernelGGL((layernorm_kernel<TI, TP, TO>), SF_LN_ARGS);
#undef SF_LN_ARGS
}

void layernorm(int dtype, int x_f32, const void *x, const void *gamma, const void *beta, float eps,
               int64_t rows, int d, void *y, hipStream_t st)
{
    if (rows <= 0) return;
    ProfScope prof(SF_KERNEL_LAYERNORM, st);
    if (dtype == SF_BF16 && !x_f32) launch_ln<h16, h16, h16>(x, gamma, beta, eps, rows, d, y, st);
    else if (dtype == SF_BF16) launch_ln<float, h16, h16>(x, gamma, beta, eps, rows, d, y, st);
    else launch_ln<float, float, float>(x, gamma, beta, eps, rows, d, y, st);
}

}  // namespace sf
