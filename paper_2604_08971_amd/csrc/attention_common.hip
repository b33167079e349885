// SentryAttend (Sec. 4.4 of the paper): the steps that are not contractions --
// K/V statistics (mean key for the sparsity score, mean value = context
// vector), the top-U query choice, the lazy-row fill -- plus the plain fp32
// kernels and the dispatch.  The bf16 MFMA kernels are in attention_bf16.hip.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "attention.hpp"
#include "gemm.hpp"
#include "topk.hpp"

namespace sf {

// ---------------------------------------------------------------- statistics
// Mean key (for the score's mean term) and mean value (context vector) over the allowed keys of a (sample, group):
//   stats[bg][0][:] = mean allowed key, stats[bg][1][:] = mean allowed value,
// and, by the block of a sample's first group, the number of allowed keys and the cleared bitmap of active rows (the
// selection that follows sets the bits of the rows it picks).  One block per (sample, group) and one launch where the
// problems fill the chip or are short (stats_parts()); else partial sums over ranges of keys and a second launch over
// them.  us, one launch / two: 1024 problems of 480 keys 26.5 / 30.6, 128 of 384 keys 7.3 / 9.3, 2 of 512 keys
// 5.8 / 9.1; 64 of 4096 keys 30.6 / 20.6.
struct StatsOut { float *stats; int32_t *n_valid; uint32_t *act_bits; };

__device__ __forceinline__ void clear_act_bits(uint32_t *act_bits, int b, int L, int nt)
{
    if (act_bits)
        for (int w = threadIdx.x; w < (L + 31) / 32; w += nt) act_bits[(int64_t)b * ((L + 31) / 32) + w] = 0u;
}

// fp32: thread t owns column e = t % DHP of both.
constexpr int STATS_NT = 512;
__global__ __launch_bounds__(STATS_NT) void kv_stats_f32_kernel(
    const float *__restrict__ K, sf_strides sk, const float *__restrict__ V, sf_strides sv, int64_t v_sj,
    int64_t v_se, const uint8_t *__restrict__ key_valid, int nG, int L, int dh, int DHP, StatsOut out,
    const int32_t *__restrict__ row0, const int32_t *__restrict__ row0_v)
{
    __shared__ float red[2][STATS_NT];
    __shared__ int red_n[STATS_NT / 64];
    const int bg = blockIdx.x, b = bg / nG, g = bg % nG;
    const int e = threadIdx.x % DHP, rg = threadIdx.x / DHP, nrg = STATS_NT / DHP;
    const float *Kb = K + sample_offset(row0, b, sk) + (int64_t)g * sk.h;
    const float *Vb = V + sample_offset(row0_v, b, sv) + (int64_t)g * sv.h;      // a transposed V is b-strided
    const uint8_t *kv = key_valid ? key_valid + (int64_t)b * L : nullptr;
    float s_k = 0.f, s_v = 0.f;
    if (e < dh)
#pragma unroll 4
        for (int j = rg; j < L; j += nrg) {
            const bool ok = !kv || kv[j];                                        // a masked row may hold anything
            const float k = Kb[(int64_t)j * sk.l + e], v = Vb[(int64_t)j * v_sj + (int64_t)e * v_se];
            s_k += ok ? k : 0.f;
            s_v += ok ? v : 0.f;
        }
    red[0][threadIdx.x] = s_k;
    red[1][threadIdx.x] = s_v;
    int c = 0;
    for (int j = threadIdx.x; j < L; j += STATS_NT) c += !kv || kv[j];
    c = block_sum<STATS_NT>(c, red_n);                                           // also orders the LDS writes
    if (g == 0) {
        if (threadIdx.x == 0) out.n_valid[b] = c;
        clear_act_bits(out.act_bits, b, L, STATS_NT);
    }
    if (threadIdx.x < DHP && e < dh) {
        float k = 0.f, v = 0.f;
        for (int r = 0; r < nrg; ++r) { k += red[0][r * DHP + e]; v += red[1][r * DHP + e]; }
        const float inv = c > 0 ? 1.0f / (float)c : 0.f;
        out.stats[(int64_t)bg * 2 * dh + e] = k * inv;
        out.stats[(int64_t)bg * 2 * dh + dh + e] = v * inv;
    }
}

// 16 bits: 16-byte loads, K rows dh-contiguous, V from its key-contiguous transposed layout [dh][Lp].  A pass covers
// NT * 8 / DH keys with one load of K and one of V per thread; UN passes are in flight while the previous UN are summed.
// NT = 256 where the problems fill the chip several times over or a block has one range of a problem, 1024 where a whole
// problem has a compute unit to itself.
template <int DH, int NT>
__global__ __launch_bounds__(NT) void kv_stats_bf16_kernel(
    const h16 *__restrict__ K, sf_strides sk, const h16 *__restrict__ VT, sf_strides svt,
    const uint8_t *__restrict__ key_valid, int nG, int L, int parts, float *__restrict__ part, StatsOut out,
    const int32_t *__restrict__ row0)
{
    constexpr int CH = DH / 8, RP = NT / CH, TPR = NT / DH, NW = NT / 64, UN = 4;
    static_assert(RP == TPR * 8 && TPR <= 64 && CH <= 64, "pass shape");
    __shared__ uint32_t words[512];                // bit j % 32 of word j / 32: key j is allowed (L <= 16384)
    __shared__ float red[NW][DH];
    __shared__ int red_n[NW];
    const int bg = blockIdx.x / parts, b = bg / nG, g = bg % nG, tid = threadIdx.x, lane = tid & 63;
    // keys [jbeg, jend) of the sample: all of them, or this block's part (a multiple of 32)
    const int range = ((L + parts - 1) / parts + 31) / 32 * 32, jbeg = blockIdx.x % parts * range, jend = min(L, jbeg + range);
    const h16 *Kb = K + sample_offset(row0, b, sk) + (int64_t)g * sk.h;
    const h16 *Vb = VT + (int64_t)b * svt.b + (int64_t)g * svt.h;        // the transposed copy: always b-strided
    const uint8_t *kv = key_valid ? key_valid + (int64_t)b * L : nullptr;

    const int r = tid / CH, c = tid % CH;          // K: row r of a pass, 16-byte chunk c
    const int e = tid / TPR, q = tid % TPR;        // V^T: row e, 8 keys at q*8 of a pass
    h16x8 kt[UN], vt[UN];
    auto fetch = [&](int j0) {
#pragma unroll
        for (int k = 0; k < UN; ++k) {
            const int jk = j0 + r + RP * k, jv = j0 + q * 8 + RP * k;
            kt[k] = h16x8{};
            vt[k] = h16x8{};
            if (jk < jend) kt[k] = *reinterpret_cast<const h16x8 *>(Kb + (int64_t)jk * sk.l + c * 8);
            if (jv < jend) vt[k] = *reinterpret_cast<const h16x8 *>(Vb + (int64_t)e * svt.l + jv);      // jv + 8 <= Lp
        }
    };
    fetch(jbeg);
    int n = 0;
    for (int j0 = jbeg; j0 < (jend + 31) / 32 * 32; j0 += NT) {         // the same trip count for every wave
        const int j = j0 + tid;
        const bool ok = j < jend && (!kv || kv[j]);
        const unsigned long long bal = __ballot(ok);
        if ((lane & 31) == 0 && j < (jend + 31) / 32 * 32) words[(j - jbeg) >> 5] = (uint32_t)(bal >> (lane & 32));
        n += ok;
    }
    n = block_sum<NT>(n, red_n);                                        // also orders the words

    float ak[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, av = 0.f;
    for (int j0 = jbeg; j0 < jend; j0 += UN * RP) {
        h16x8 kc[UN], vc[UN];
#pragma unroll
        for (int k = 0; k < UN; ++k) { kc[k] = kt[k]; vc[k] = vt[k]; }
        if (j0 + UN * RP < jend) fetch(j0 + UN * RP);
        // validity is a select: masked rows may hold anything
#pragma unroll
        for (int k = 0; k < UN; ++k) {
            const int jk = j0 + r + RP * k, jv = j0 + q * 8 + RP * k;
            const bool ok = jk < jend && ((words[(jk - jbeg) >> 5] >> (jk & 31)) & 1u);
            const uint32_t bits = jv < jend ? words[(jv - jbeg) >> 5] >> (jv & 31) : 0u;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                ak[t] += ok ? (float)kc[k][t] : 0.f;
                av += ((bits >> t) & 1u) ? (float)vc[k][t] : 0.f;
            }
        }
    }
    // K: rows of a wave by shuffles, then the waves; V: the lanes of a row
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int o = CH; o < 64; o <<= 1) ak[t] += __shfl_xor(ak[t], o);
    if (lane < CH) {
#pragma unroll
        for (int t = 0; t < 8; ++t) red[tid >> 6][lane * 8 + t] = ak[t];
    }
#pragma unroll
    for (int o = 1; o < TPR; o <<= 1) av += __shfl_xor(av, o);
    const float inv = parts > 1 ? 1.0f : n > 0 ? 1.0f / (float)n : 0.f;
    float *st = parts > 1 ? part + (int64_t)blockIdx.x * (2 * DH + 1) : out.stats + (int64_t)bg * 2 * DH;
    if (q == 0) st[DH + e] = av * inv;
    __syncthreads();
    if (tid < DH) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += red[w][tid];
        st[tid] = s * inv;
    }
    if (parts > 1) {
        if (tid == 0) st[2 * DH] = (float)n;
    } else if (g == 0) {
        if (tid == 0) out.n_valid[b] = n;
        clear_act_bits(out.act_bits, b, L, NT);
    }
}

// Latency is all there is: the counts are one load per thread, and 256 / (2 dh) threads share a column's ranges (one after the
// other, counts first, 128 ranges of dh 32 took 10 us longer).
__global__ __launch_bounds__(256) void kv_stats_sum_kernel(const float *__restrict__ part, int parts, int nG, int L, int dh,
                                                           StatsOut out)
{
    __shared__ float red[256];
    __shared__ int red_n[4];
    const int bg = blockIdx.x, b = bg / nG, cols = 2 * dh, share = 256 / cols;       // dh 32, 64 or 128
    const int t = threadIdx.x % cols, first = threadIdx.x / cols;
    const float *p = part + (int64_t)bg * parts * (cols + 1);
    int n = 0;
    for (int c = threadIdx.x; c < parts; c += 256) n += (int)p[(int64_t)c * (cols + 1) + cols];
    float s = 0.f;
#pragma unroll 8
    for (int c = first; c < parts; c += share) s += p[(int64_t)c * (cols + 1) + t];
    red[threadIdx.x] = s;
    n = block_sum<256>(n, red_n);                                                    // also orders the LDS writes
    if (first == 0) {
        for (int k = 1; k < share; ++k) s += red[k * cols + t];
        out.stats[(int64_t)bg * cols + t] = s * (n > 0 ? 1.0f / (float)n : 0.f);
    }
    if (bg % nG == 0) {
        if (threadIdx.x == 0) out.n_valid[b] = n;
        clear_act_bits(out.act_bits, b, L, 256);
    }
}

// Ranges of keys per problem: one where there are twice as many problems as compute units, or at most 1024 keys of 64 KB
// (8 problems of 1024 keys, dh 128: 35.6 us for the whole call with one range, 29.9 with eight; 2048 keys, dh 32: 24.5 / 22.3);
// else towards 1024 blocks of at least 128 keys.
static int stats_parts(int64_t problems, int L, int dh)
{
    if (problems >= 512 || (L <= 1024 && L * dh <= 65536)) return 1;
    return (int)std::min<int64_t>(ceil_div(L, 128), (1024 + problems - 1) / problems);
}

// ------------------------------------------------------------------- lazy rows
// Every row that is not active in a head takes the head's group's context vector there: done by the block that has just
// chosen the head's active rows (it needs no row -> slot map from memory), before the active pass writes those rows.
// O == NULL: somebody else does (fill_rows_kernel, or a caller that projects the lazy rows itself).  us, selection + fill in two launches / in one: 1024 rows of 480
// scores 10.3 + 22.7 / 18.7 (63 MB written), 768 rows of 512 8.8 + 18.0 / 15.6, 384 rows of 384 7.4 + 7.0 / 9.0.
template <class T>
struct Fill {
    T *O; int64_t ldo;
    const float *stats; const int32_t *head_group; int hg_stride; const int32_t *pattern_id; int nG, dh;
    const int32_t *row0, *ext;
    const float *part; int parts;      // or NULL: the context vector is the sum of `parts` pieces [B*nG, parts, dh] over the allowed keys
};

// The thread's share of the context vector (VEC consecutive elements), read ahead of the selection, and the rows it writes:
// kept[i] != 0: row i < L is active.  Packed samples also own the padding rows behind their tokens (ext[b] >= the
// sample's length; rows at or beyond L are padding).  PART: the context vector follows with mean_of().
template <int NT, int VEC, class T, bool PART = false>
struct HeadFill {
    typedef __attribute__((ext_vector_type(VEC))) T vec;
    vec v;
    T *o;
    int rows, step;
    __device__ __forceinline__ HeadFill(const Fill<T> &f, int b, int h, int L) : o(nullptr)
    {
        const int qv = f.dh / VEC, c = threadIdx.x % qv;
        step = NT / qv;
        if (!f.O || (int)threadIdx.x >= step * qv) return;
        rows = f.ext ? f.ext[b] : L;
        if constexpr (!PART) {
            const float *ctx = f.stats + (((int64_t)b * f.nG + group(f, b, h)) * 2 + 1) * f.dh + c * VEC;
#pragma unroll
            for (int t = 0; t < VEC; ++t) v[t] = from_f32<T>(ctx[t]);
        }
        o = f.O + sample_row(f.row0, b, L) * f.ldo + (int64_t)h * f.dh + c * VEC;
    }
    static __device__ __forceinline__ int group(const Fill<T> &f, int b, int h)
    {
        return f.head_group[(int64_t)(f.pattern_id ? f.pattern_id[b] : 0) * f.hg_stride + h];
    }
    // the context vector from its sum over n allowed keys (dh values in LDS)
    __device__ __forceinline__ void mean_of(const Fill<T> &f, const float *sum, int n)
    {
        const float inv = n > 0 ? 1.0f / (float)n : 0.f;
        const int c = threadIdx.x % (f.dh / VEC);
#pragma unroll
        for (int t = 0; t < VEC; ++t) v[t] = from_f32<T>(sum[c * VEC + t] * inv);
    }
    __device__ __forceinline__ void put(const Fill<T> &f, int r) const { *reinterpret_cast<vec *>(o + (int64_t)r * f.ldo) = v; }
    __device__ __forceinline__ void write(const Fill<T> &f, int L, const uint32_t *kept) const
    {
        if (!o) return;
#pragma unroll 4
        for (int r = threadIdx.x / (f.dh / VEC); r < rows; r += step)
            if (r >= L || !kept[r]) put(f, r);
    }
};

// Every row of a head, by many blocks: the active pass, which comes later, writes the active ones over it.
template <int VEC, class T>
__global__ __launch_bounds__(256) void fill_rows_kernel(int nH, int L, Fill<T> fill)
{
    const HeadFill<256, VEC, T> hf(fill, blockIdx.y / nH, blockIdx.y % nH, L);
    if (!hf.o) return;
#pragma unroll 4
    for (int r = blockIdx.x * hf.step + threadIdx.x / (fill.dh / VEC); r < hf.rows; r += gridDim.x * hf.step) hf.put(fill, r);
}

// ------------------------------------------------------------------- selection
// One block per (b, head): the U_eff = min(U, u_active[b], #allowed) queries with the
// highest score, ties to the lower index; emitted ascending.  score == NULL
// means "every allowed query" (used when U >= L).  The score may come in n > 1 ranges of keys, as n planes of largest
// products and one of products with the mean key (`stride` apart): the score is (largest of all - mean) * scale, 0 for a
// sample without a key to score by (n_keys), and `out` then receives it.
struct ScoreParts { const float *score; int64_t stride; int n, H; const int32_t *n_keys; float scale; float *out; int outH; };     // H: heads per sample

// PART: fill.part is there, in an instance of its own (a call without it waited for the context vector where it asked: 0.1 to 0.3 us).
template <int NT, int VEC, class T, bool PART>
__global__ __launch_bounds__(NT) void select_kernel(
    ScoreParts sc, const uint8_t *__restrict__ key_valid, int nH, int L,
    int U, const int32_t *__restrict__ u_active, int32_t *__restrict__ sel, int selH, int32_t *__restrict__ slot,
    uint32_t *__restrict__ act_bits, Fill<T> fill)
{
    extern __shared__ uint32_t keys[];
    __shared__ __attribute__((aligned(16))) int scratch[TOPK_SCRATCH];
    __shared__ int red[NT / 64];    // not part of `scratch`: block_topk clears its histograms there right away
    const int bh = blockIdx.x, b = bh / nH, h = bh % nH;
    const uint8_t *kv = key_valid ? key_valid + (int64_t)b * L : nullptr;
    const int64_t m0 = ((int64_t)b * sc.H + h) * L;
    int32_t *sl = slot ? slot + (int64_t)bh * L : nullptr;      // only the active-row projection reads it
    int32_t *se = sel + ((int64_t)b * selH + h) * U;
    HeadFill<NT, VEC, T, PART> hf(fill, b, h, L);
    __shared__ float ctx[PART ? 256 : 1];
    if (PART && threadIdx.x < fill.dh) {                        // with a key mask only: its count orders these writes
        const float *p = fill.part + ((int64_t)b * fill.nG + hf.group(fill, b, h)) * fill.parts * fill.dh + threadIdx.x;
        // in eight chains: one of 28 (1777 keys of mean 1) errs by 6.8e-8 of the sum, these by 2.9e-8, the statistics launch by 4.9e-8
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int i = 0; i < fill.parts; i += 8) {
#pragma unroll
            for (int k = 0; k < 8; ++k) s[k] += i + k < fill.parts ? p[(int64_t)(i + k) * fill.dh] : 0.f;
        }
        ctx[threadIdx.x] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    }
    const bool no_key = sc.n > 1 && sc.n_keys[b] == 0;
    int c = 0;
    for (int i = threadIdx.x; i < L; i += NT) {
        const bool ok = !kv || kv[i];
        // allowed queries get a key >= 1 (the smallest, of a NaN with every bit set, is 0 by the map), others key 0
        uint32_t key = 1u;
        if (sc.score) {
            float m = sc.score[m0 + i];
            if (sc.n > 1) {
                const float mean = sc.score[sc.n * sc.stride + m0 + i];
#pragma unroll 4
                for (int p = 1; p < sc.n; ++p) m = fmaxf(m, sc.score[p * sc.stride + m0 + i]);
                m = !ok ? -INFINITY : no_key ? 0.f : (m - mean) * sc.scale;
                if (sc.out) sc.out[((int64_t)b * sc.outH + h) * L + i] = m;
            }
            key = max(sortable_key(m), 1u);
        }
        keys[i] = ok ? key : 0u;
        c += ok;
    }
    const int n_ok = kv ? block_sum<NT>(c, red) : L;
    if constexpr (PART) hf.mean_of(fill, ctx, n_ok);
    // u_active: this sample's own number of active queries (samples of different length in one batch)
    const int k = min(u_active ? min(max(u_active[b], 0), U) : U, n_ok);
    if (k == 0) {
        __syncthreads();
        for (int i = threadIdx.x; i < L; i += NT) {
            keys[i] = 0u;
            if (sl) sl[i] = -1;
        }
    } else {
        auto emit = [&](int i, bool kept, int pos) {
            keys[i] = kept ? 1u : 0u;
            if (sl) sl[i] = kept ? pos : -1;
            if (kept) {
                se[pos] = i;
                if (act_bits) atomicOr(&act_bits[(int64_t)b * ((L + 31) / 32) + (i >> 5)], 1u << (i & 31));
            }
        };
        if (L <= NT) block_topk<NT, 1>(keys, L, k, scratch, k == n_ok, emit);
        else if (L <= NT * 4) block_topk<NT, 4>(keys, L, k, scratch, k == n_ok, emit);
        else block_topk<NT>(keys, L, k, scratch, k == n_ok, emit);
    }
    for (int r = k + threadIdx.x; r < U; r += NT) se[r] = -1;
    __syncthreads();
    hf.write(fill, L, keys);
}

// Caller-supplied active set: the same outputs from its list.
template <int VEC, class T>
__global__ __launch_bounds__(256) void forced_slot_kernel(const int32_t *__restrict__ forced, int forcedH,
                                                          int nH, int L, int U, int32_t *__restrict__ sel,
                                                          int selH, int32_t *__restrict__ slot,
                                                          uint32_t *__restrict__ act_bits, Fill<T> fill)
{
    extern __shared__ uint32_t kept[];
    const int bh = blockIdx.x, b = bh / nH, h = bh % nH;
    int32_t *sl = slot ? slot + (int64_t)bh * L : nullptr;
    const HeadFill<256, VEC, T> hf(fill, b, h, L);
    for (int i = threadIdx.x; i < L; i += 256) {
        kept[i] = 0u;
        if (sl) sl[i] = -1;
    }
    __syncthreads();
    for (int r = threadIdx.x; r < U; r += 256) {
        int q = forced[((int64_t)b * forcedH + h) * U + r];
        if (q < 0 || q >= L) q = -1;
        sel[((int64_t)b * selH + h) * U + r] = q;
        if (q >= 0) {
            kept[q] = 1u;
            if (sl) sl[q] = r;
            if (act_bits) atomicOr(&act_bits[(int64_t)b * ((L + 31) / 32) + (q >> 5)], 1u << (q & 31));
        }
    }
    __syncthreads();
    hf.write(fill, L, kept);
}

// Merge of the key splits of the active pass: one wave per (sample, head,
// active slot).  Lane sp holds the (max, sum) pair of split sp (splits <= 64),
// the weights 2^(m_sp - m) are formed once, then lane e accumulates output
// dimension e over the splits (partials are [b, head, split, slot, dh]).
template <class T>
__global__ __launch_bounds__(256) void merge_splits_kernel(
    int nH, int L, int dh, int U, int Upad, int splits, int64_t n_waves, const int32_t *__restrict__ sel,
    int selH, const float *__restrict__ part_o, const float *__restrict__ part_ml, T *__restrict__ O,
    int64_t ldo, const int32_t *__restrict__ row0)
{
    const int lane = threadIdx.x & 63;
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w >= n_waves) return;
    const int s = (int)(w % U);
    const int64_t bh = w / U;
    const int h = (int)(bh % nH);
    const int64_t b = bh / nH;
    const int64_t base = bh * splits;
    // an empty slot (fewer allowed queries than U) has no row and no partials: nothing to merge
    const int qi = sel[((int64_t)b * selH + h) * U + s];
    if (qi < 0) return;                                     // wave-uniform
    float ms = -INFINITY, ls = 0.f;
    if (lane < splits) {
        const int64_t q = (base + lane) * Upad + s;
        ms = part_ml[q * 2];
        ls = part_ml[q * 2 + 1];
    }
    float m = ms;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    const float wgt = (ms == -INFINITY) ? 0.f : exp2f(ms - m);
    float den = wgt * ls;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) den += __shfl_xor(den, o);
    const float inv = den > 0.f ? 1.0f / den : 0.f;
    T *orow = O + (sample_row(row0, (int)b, L) + qi) * ldo + (int64_t)h * dh;
    for (int e = lane; e < dh; e += 64) {
        float acc = 0.f;
        const float *po = part_o + (base * Upad + s) * dh + e;
#pragma unroll 4
        for (int sp = 0; sp < splits; ++sp) acc += __shfl(wgt, sp) * po[(int64_t)sp * Upad * dh];
        orow[e] = from_f32<T>(acc * inv);
    }
}

// V [B,nG,L,dh] -> VT [B,nG,dh,Lp] (bf16), 32x32 tiles through LDS.
__global__ __launch_bounds__(256) void transpose_v_kernel(const uint16_t *__restrict__ V, sf_strides sv, int nG,
                                                          int L, int dh, int Lp, uint16_t *__restrict__ VT,
                                                          const int32_t *__restrict__ row0)
{
    __shared__ uint16_t tile[32][33];
    const int bg = blockIdx.z, b = bg / nG, g = bg % nG;
    const int j0 = blockIdx.x * 32, e0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const uint16_t *Vb = V + sample_offset(row0, b, sv) + (int64_t)g * sv.h;
    for (int jj = ty; jj < 32; jj += 8) {
        const int j = j0 + jj, e = e0 + tx;
        tile[jj][tx] = (j < L && e < dh) ? Vb[(int64_t)j * sv.l + e] : (uint16_t)0;
    }
    __syncthreads();
    uint16_t *o = VT + (int64_t)bg * dh * Lp;
    for (int ee = ty; ee < 32; ee += 8) {
        const int e = e0 + ee, j = j0 + tx;
        if (e < dh && j < Lp) o[(int64_t)e * Lp + j] = tile[tx][ee];
    }
}

// ------------------------------------------------------------ plain fp32 path
// Sparsity score over the Lk keys of K (validity key_mask [B,Lk] or NULL, n_keys[b] of them valid): the sample's own
// keys, or the gathered key sample.  A block serves SF32_TQ queries of one (sample, head): 16 threads per query, each with
// every 16th key of the tile that the block has staged in LDS; a key's products are summed in the order of e, the keys of a
// query over its 16 threads.  What bounds it on the small models it is there for is the chain of dependent steps: one
// thread per query walked all keys from memory, 45 us for 2 samples of 48 tokens; 5.7 us now.
constexpr int SF32_TQ = 16, SF32_TK = 32;
__global__ __launch_bounds__(256) void score_f32_kernel(
    const float *__restrict__ Q, sf_strides sq, const float *__restrict__ K, sf_strides sk,
    const int32_t *__restrict__ head_group, int hg_stride, const int32_t *__restrict__ pattern_id,
    const uint8_t *__restrict__ query_valid, const uint8_t *__restrict__ key_mask,
    const int32_t *__restrict__ n_keys, int nH, int L, int Lk, int dh, float *__restrict__ score, int scoreH,
    const int32_t *__restrict__ row0, int keys_packed)
{
    extern __shared__ float s32[];                          // [SF32_TQ + SF32_TK][dh + 1]
    const int bh = blockIdx.y, b = bh / nH, h = bh % nH, tid = threadIdx.x;
    const int qi = tid >> 4, kl = tid & 15, ldt = dh + 1;
    const int i0 = blockIdx.x * SF32_TQ, i = i0 + qi;
    const int nk = n_keys[b];
    const uint8_t *km = key_mask ? key_mask + (int64_t)b * Lk : nullptr;
    const int g = head_group[(int64_t)(pattern_id ? pattern_id[b] : 0) * hg_stride + h];
    const float *Qb = Q + sample_offset(row0, b, sq) + (int64_t)h * sq.h;
    // the gathered key sample lives in the workspace and is b-strided whatever the layout of K
    const float *Kb = K + sample_offset(keys_packed ? row0 : nullptr, b, sk) + (int64_t)g * sk.h;
    float *qs = s32, *ks = s32 + SF32_TQ * ldt;
    for (int c = tid; c < SF32_TQ * dh; c += 256) {
        const int r = c / dh, e = c - r * dh;
        qs[r * ldt + e] = i0 + r < L ? Qb[(int64_t)(i0 + r) * sq.l + e] : 0.f;
    }
    const float scale = 1.0f / sqrtf((float)dh);
    float mx = -INFINITY, sum = 0.f;
    for (int j0 = 0; j0 < Lk && nk > 0; j0 += SF32_TK) {    // nk is the sample's: uniform over the block
        const int nt = min(SF32_TK, Lk - j0);
        for (int c = tid; c < nt * dh; c += 256) {
            const int r = c / dh, e = c - r * dh;
            ks[r * ldt + e] = Kb[(int64_t)(j0 + r) * sk.l + e];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < SF32_TK / 16; ++u) {
            const int r = kl + u * 16;
            if (r >= nt || (km && !km[j0 + r])) continue;
            const float *q = qs + qi * ldt, *k = ks + r * ldt;
            float s = 0.f;
            for (int e = 0; e < dh; ++e) s = fmaf(q[e], k[e], s);
            s *= scale;
            mx = fmaxf(mx, s);
            sum += s;
        }
        __syncthreads();
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
        mx = fmaxf(mx, __shfl_xor(mx, o));
        sum += __shfl_xor(sum, o);
    }
    if (kl != 0 || i >= L) return;
    float *out = score + ((int64_t)b * scoreH + h) * L + i;
    if (query_valid && !query_valid[(int64_t)b * L + i]) *out = -INFINITY;
    else *out = nk == 0 ? 0.f : mx - sum / (float)nk;
}

// Key sample of the sparsity score: one block per (sample, group).  The sample is treated as a set
// (LDS bit words, integer atomics), intersected with the allowed keys, listed in ascending key order
// and gathered into Ks [B,nG,Sp,dh] (zero rows beyond the n_keys[b] listed keys), with the row validity
// ks_valid [B,Sp] and the mean listed key in ks_stats [(b*nG+g)*2*dh + e] (the layout of the K/V
// statistics; only the mean-key half is used).
template <class T>
__global__ __launch_bounds__(256) void gather_key_sample_kernel(
    const T *__restrict__ K, sf_strides sk, const uint8_t *__restrict__ key_valid,
    const int32_t *__restrict__ sample_idx, int n_sample, int nG, int L, int dh, int Sp,
    T *__restrict__ Ks, uint8_t *__restrict__ ks_valid, float *__restrict__ ks_stats,
    int32_t *__restrict__ n_keys, const int32_t *__restrict__ row0)
{
    extern __shared__ uint32_t gsm[];
    const int nwords = (L + 31) / 32;
    uint32_t *words = gsm;                                        // [nwords]
    int32_t *list = reinterpret_cast<int32_t *>(gsm + nwords);    // [Sp]
    __shared__ int nk_s;
    const int bg = blockIdx.x, b = bg / nG, g = bg % nG, tid = threadIdx.x;
    const uint8_t *kv = key_valid ? key_valid + (int64_t)b * L : nullptr;
    for (int w = tid; w < nwords; w += 256) words[w] = 0u;
    __syncthreads();
    for (int r = tid; r < n_sample; r += 256) {
        const int idx = sample_idx[(int64_t)b * n_sample + r];
        if (idx >= 0 && idx < L && (!kv || kv[idx])) atomicOr(&words[idx >> 5], 1u << (idx & 31));
    }
    __syncthreads();
    if (tid < 64) {                                               // ascending list of the set bits
        int base = 0;
        for (int w0 = 0; w0 < nwords; w0 += 64) {
            uint32_t w = (w0 + tid < nwords) ? words[w0 + tid] : 0u;
            const int pc = __popc(w);
            int incl = pc;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_up(incl, o);
                if (tid >= o) incl += t;
            }
            int pos = base + incl - pc;
            while (w) {
                const int bit = __ffs((int)w) - 1;
                list[pos++] = (w0 + tid) * 32 + bit;
                w &= w - 1u;
            }
            base += __shfl(incl, 63);
        }
        if (tid == 0) nk_s = base;
    }
    __syncthreads();
    const int nk = nk_s;                                          // <= n_sample <= Sp
    const T *Kb = K + sample_offset(row0, b, sk) + (int64_t)g * sk.h;
    T *out = Ks + (int64_t)bg * Sp * dh;
    for (int t = tid; t < Sp * dh; t += 256) {
        const int r = t / dh, e = t % dh;
        out[t] = r < nk ? Kb[(int64_t)list[r] * sk.l + e] : from_f32<T>(0.f);
    }
    if (g == 0) {
        for (int r = tid; r < Sp; r += 256) ks_valid[(int64_t)b * Sp + r] = r < nk ? 1 : 0;
        if (tid == 0) n_keys[b] = nk;
    }
    for (int e = tid; e < dh; e += 256) {
        float acc = 0.f;
        for (int r = 0; r < nk; ++r) acc += to_f32(Kb[(int64_t)list[r] * sk.l + e]);
        ks_stats[((int64_t)bg * 2) * dh + e] = nk ? acc / (float)nk : 0.f;
    }
}

// Active rows, Eq. (6): one 64-lane wave per (b, head, slot).
__global__ __launch_bounds__(64) void attend_f32_kernel(
    const float *__restrict__ Q, sf_strides sq, const float *__restrict__ K, sf_strides sk,
    const float *__restrict__ V, sf_strides sv, int64_t v_sj, int64_t v_se,
    const int32_t *__restrict__ head_group, int hg_stride, const int32_t *__restrict__ pattern_id,
    const uint8_t *__restrict__ key_valid, const int32_t *__restrict__ sel, int selH, int nH, int L, int dh,
    int U, float *__restrict__ O, int64_t ldo, const int32_t *__restrict__ row0)
{
    extern __shared__ float prob[];
    const int bh = blockIdx.y, b = bh / nH, h = bh % nH, lane = threadIdx.x;
    const int qi = sel[((int64_t)b * selH + h) * U + blockIdx.x];
    if (qi < 0) return;
    const uint8_t *kv = key_valid ? key_valid + (int64_t)b * L : nullptr;
    const int g = head_group[(int64_t)(pattern_id ? pattern_id[b] : 0) * hg_stride + h];
    const float *q = Q + sample_offset(row0, b, sq) + (int64_t)h * sq.h + (int64_t)qi * sq.l;
    const float *Kb = K + sample_offset(row0, b, sk) + (int64_t)g * sk.h;
    const float *Vb = V + sample_offset(row0, b, sv) + (int64_t)g * sv.h;
    const float scale = 1.0f / sqrtf((float)dh);
    float mx = -INFINITY;
    for (int j = lane; j < L; j += 64) {
        float s = -INFINITY;
        if (!kv || kv[j]) {
            const float *k = Kb + (int64_t)j * sk.l;
            s = 0.f;
            for (int e = 0; e < dh; ++e) s = fmaf(q[e], k[e], s);
            s *= scale;
        }
        prob[j] = s;
        mx = fmaxf(mx, s);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    float den = 0.f;
    for (int j = lane; j < L; j += 64) {
        const float pj = prob[j] == -INFINITY ? 0.f : expf(prob[j] - mx);
        prob[j] = pj;
        den += pj;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) den += __shfl_xor(den, o);
    __syncthreads();
    const float inv = 1.0f / den;
    // narrow heads: the keys are dealt to the 64 / w groups of w lanes that a row of V needs
    int w = 64;
    while (w / 2 >= dh) w >>= 1;
    for (int e0 = 0; e0 < dh; e0 += w) {
        const int e = e0 + (lane & (w - 1));
        const float *v = Vb + (int64_t)min(e, dh - 1) * v_se;
        float acc = 0.f;
#pragma unroll 4
        for (int j = lane / w; j < L; j += 64 / w) acc = fmaf(prob[j], v[(int64_t)j * v_sj], acc);
        for (int o = w; o < 64; o <<= 1) acc += __shfl_xor(acc, o);
        if (lane < w && e < dh) O[(sample_row(row0, b, L) + qi) * ldo + (int64_t)h * dh + e] = acc * inv;
    }
}

// ------------------------------------------------------------------- planning
static AttnPlan attn_plan_parts(int dtype, const AttnArgs &a, void *ws, int score_parts)
{
    AttnPlan pl{};
    const bool sparse = a.U < a.L;
    pl.Upad = (int)align_up(a.U > 0 ? a.U : 1, 32);
    pl.Lp = (int)align_up(a.L, 8);
    pl.Sp = a.n_sample > 0 ? (int)align_up(a.n_sample, 64) : 0;
    pl.splits = 1;
    pl.keys_per_split = (int)align_up(a.L, 64);
    if (dtype == SF_BF16 && a.U > 0) {
        // the staged active pass has only B*nG independent (sample, group) problems: with fewer than one per compute unit
        // the keys are split until one workgroup per compute unit exists (256), and only into pieces of at least four key tiles:
        // two fit a compute unit, but the parts of a split are joined.  Of 110 calls of 1100 to 16384 keys, 13 are split more
        // with a target of 384 or 512: 1.01 of the time (0.94 to 1.09 either way)
        const int64_t bg = (int64_t)a.B * a.nG;
        int want = bg >= 256 || !sparse ? 1 : (int)((256 + bg - 1) / bg);
        const int max_splits = a.L / 256 > 0 ? a.L / 256 : 1;
        if (want > max_splits) want = max_splits;
        if (want > 64) want = 64;                     // the merge holds one split per lane
        const int keys = (int)align_up(ceil_div(a.L, want), 64), splits = ceil_div(a.L, keys);
        pl.staged = attend_bf16_staged(a, splits);
        if (pl.staged) { pl.splits = splits; pl.keys_per_split = keys; }
    }
    pl.score_parts = score_parts;
    Carver c(ws);
    const size_t BH = (size_t)a.B * a.nH, BG = (size_t)a.B * a.nG;
    pl.vt = (dtype == SF_BF16 && !a.v_transposed) ? c.take<uint16_t>(BG * a.dh * pl.Lp) : nullptr;
    pl.stat_parts = dtype == SF_BF16 ? stats_parts(BG, a.L, a.dh) : 1;
    pl.stat_part = pl.stat_parts > 1 ? c.take<float>(BG * pl.stat_parts * (2 * a.dh + 1)) : nullptr;
    pl.stats = c.take<float>(BG * 2 * a.dh);
    pl.n_valid = c.take<int32_t>(a.B);
    pl.score = c.take<float>(BH * a.L * (pl.score_parts > 1 ? pl.score_parts + 1 : 1));
    pl.sel = c.take<int32_t>(BH * (a.U > 0 ? a.U : 1));
    pl.slot = a.need_slot ? c.take<int32_t>(BH * a.L) : nullptr;
    if (pl.splits > 1) {
        pl.part_o = c.take<float>(BH * pl.Upad * pl.splits * a.dh);
        pl.part_ml = c.take<float>(BH * pl.Upad * pl.splits * 2);
    }
    if (pl.Sp > 0) {
        pl.ks = c.take<char>(BG * pl.Sp * a.dh * elem_size(dtype));
        pl.ks_valid = c.take<uint8_t>((size_t)a.B * pl.Sp);
        pl.ks_stats = c.take<float>(BG * 2 * a.dh);
        pl.n_keys = c.take<int32_t>(a.B);
    }
    pl.bytes = c.off;
    return pl;
}

// The score stream is split into key ranges only where the workspace has room for their planes (the score is the same
// either way): a caller's or the built-in buffer that holds everything else is large enough.
AttnPlan attn_plan(int dtype, const AttnArgs &a, void *ws)
{
    const bool sparse = a.U > 0 && a.U < a.L;
    const int parts = dtype == SF_BF16 && sparse ? score_bf16_parts(a, a.n_sample > 0 ? (int)align_up(a.n_sample, 64) : a.L) : 1;
    AttnPlan pl = attn_plan_parts(dtype, a, ws, parts);
    if (parts > 1 && a.ws_bytes > 0 && pl.bytes > a.ws_bytes) pl = attn_plan_parts(dtype, a, ws, 1);
    return pl;
}

int32_t attention_forward(int dtype, const AttnArgs &a, hipStream_t st)
{
    if (a.B <= 0) return SF_OK;
    if (a.L > 16384) return fail(SF_ERR_SHAPE, "sparse_gqa: L <= 16384 required");
    if (a.dh % 4 || a.ldo % 4) return fail(SF_ERR_SHAPE, "sparse_gqa: dh and ldo must be multiples of 4");
    if (dtype == SF_BF16) {
        if (a.dh != 32 && a.dh != 64 && a.dh != 128)
            return fail(SF_ERR_SHAPE, "sparse_gqa(bf16): dh must be 32, 64 or 128");
        if ((a.sq.b | a.sq.h | a.sq.l | a.sk.b | a.sk.h | a.sk.l | a.sv.b | a.sv.h | a.sv.l) % 8)
            return fail(SF_ERR_SHAPE, "sparse_gqa(bf16): strides must be multiples of 8 elements");
    } else if (a.dh > 256) {
        return fail(SF_ERR_SHAPE, "sparse_gqa(f32): dh <= 256 required");
    }
    // limits of the bf16 launchers (their 1-D grids), checked here so that nothing is enqueued when they fail
    if (dtype == SF_BF16 && a.nH > 64) return fail(SF_ERR_SHAPE, "sparse_gqa(bf16): at most 64 heads");
    if ((int64_t)a.B * a.nH * ceil_div(a.L, 32) * 64 > ((int64_t)1 << 30))
        return fail(SF_ERR_SHAPE, "sparse_gqa: too many work items (B * heads * L / 32 must stay below 2^24)");
    AttnPlan pl = attn_plan(dtype, a, a.ws);
    if (pl.bytes > 0 && (!a.ws || a.ws_bytes < pl.bytes || ((uintptr_t)a.ws & 255)))
        return fail(SF_ERR_WORKSPACE, "sparse_gqa: workspace of %zu bytes (256-byte aligned) required, got %zu",
                    pl.bytes, a.ws_bytes);

    const int BH = a.B * a.nH, BG = a.B * a.nG;
    // V as the kernels will read it
    const void *Vuse = a.V;
    sf_strides svu = a.sv;
    int vT = a.v_transposed;
    // Every allowed query active: no score asks for the mean key, and the context vector of the masked rows is summed from what the
    // transposition of V leaves per 64 tokens (in the place of the score) by the blocks that write those rows.
    VSums sums{};
    if (a.U >= a.L && a.key_valid && !a.forced_sel && !a.act_bits && !a.skip_fill &&
        (int64_t)BG * ceil_div(pl.Lp, 64) * a.dh <= (int64_t)BH * a.L)
        sums = VSums{a.key_valid, a.nG, a.dh, pl.score};
    bool summed = false;
    if (dtype == SF_BF16 && !a.v_transposed) {
        // whole chunks of 16 bytes where V is packed head by head or token by token (8 samples of 1777 keys, 4 groups of dh 64:
        // 9.2 us, 6.7 so), else element by element
        const bool whole = (uintptr_t)a.V % 16 == 0 && !a.row0;
        if (whole && a.sv.h == a.L * a.sv.l && a.sv.b == a.nG * a.sv.h) {
            transpose_v(a.V, a.sv.l, 0, a.dh, BG, a.L, pl.Lp, pl.vt, st, nullptr, sums);
            summed = sums.part != nullptr;
        } else if (whole && a.sv.h == a.dh && a.sv.b == a.L * a.sv.l) {
            transpose_v(a.V, a.sv.l, 0, a.nG * a.dh, a.B, a.L, pl.Lp, pl.vt, st, nullptr, sums);
            summed = sums.part != nullptr;
        } else {
            dim3 grid(ceil_div(pl.Lp, 32), ceil_div(a.dh, 32), BG);
            hipLaunchKernelGGL(transpose_v_kernel, grid, dim3(256), 0, st, (const uint16_t *)a.V, a.sv, a.nG,
                               a.L, a.dh, pl.Lp, (uint16_t *)pl.vt, a.row0);
        }
        Vuse = pl.vt;
        svu.b = (int64_t)a.nG * a.dh * pl.Lp;
        svu.h = (int64_t)a.dh * pl.Lp;
        svu.l = pl.Lp;
        vT = 1;
    }
    const int64_t v_sj = vT ? 1 : svu.l, v_se = vT ? svu.l : 1;

    if (dtype == SF_BF16 && attend_short(a) && !a.forced_sel && !a.skip_fill && !a.act_bits && a.ldo % 8 == 0 &&
        (uintptr_t)a.O % 16 == 0) {
        if (int32_t rc = attend_short_bf16(a, Vuse, svu, pl.Lp, st)) return rc;
        return check_launch("sparse_gqa_forward");
    }

    if (dtype == SF_F32 && attend_short_f32(a) && !a.forced_sel && !(a.sample_idx && pl.Sp > 0) && !a.skip_fill && !a.act_bits &&
        (uintptr_t)a.O % 16 == 0) {
        if (int32_t rc = attend_short_f32_run(a, st)) return rc;
        return check_launch("sparse_gqa_forward");
    }

    // 1. statistics: mean key (for the score's mean term) and context vector; nobody asks for them where every row is active
    // and the choice is not the caller's
    const bool all_active = a.U >= a.L && !a.key_valid && !a.forced_sel && !a.act_bits && !a.skip_fill && !a.row0;
    if (!all_active && !summed) {
        const StatsOut so{pl.stats, pl.n_valid, a.act_bits};
        if (dtype == SF_BF16) {
            const int parts = pl.stat_parts;
            const bool many = parts > 1 || BG >= 512;
#define SF_STATS_ARGS 0, st, (const h16 *)a.K, a.sk, (const h16 *)Vuse, svu, a.key_valid, a.nG, a.L, parts, pl.stat_part, so, a.row0
#define SF_STATS_LAUNCH(DH)                                                                                         \
    do {                                                                                                            \
        if (many) hipLaunchKernelGGL((kv_stats_bf16_kernel<DH, 256>), dim3(BG * parts), dim3(256), SF_STATS_ARGS);  \
        else hipLaunchKernelGGL((kv_stats_bf16_kernel<DH, 1024>), dim3(BG * parts), dim3(1024), SF_STATS_ARGS);     \
    } while (0)
            if (a.dh == 32) SF_STATS_LAUNCH(32);
            else if (a.dh == 64) SF_STATS_LAUNCH(64);
            else SF_STATS_LAUNCH(128);
#undef SF_STATS_LAUNCH
#undef SF_STATS_ARGS
            if (parts > 1)
                hipLaunchKernelGGL(kv_stats_sum_kernel, dim3(BG), dim3(256), 0, st, pl.stat_part, parts, a.nG, a.L, a.dh, so);
        } else {
            int DHP = 4;
            while (DHP < a.dh) DHP *= 2;
            hipLaunchKernelGGL(kv_stats_f32_kernel, dim3(BG), dim3(STATS_NT), 0, st, (const float *)a.K, a.sk,
                               (const float *)Vuse, svu, v_sj, v_se, a.key_valid, a.nG, a.L, a.dh, DHP, so, a.row0,
                               vT ? nullptr : a.row0);
        }
    }

    // 2. active set, and the lazy rows of every head
    const int userH = a.selH > 0 ? a.selH : a.nH;
    int32_t *sel = a.sel_out ? a.sel_out : pl.sel;
    const int selH = a.sel_out ? userH : a.nH;
    // the row -> slot map is read by the projection of the active rows only
    int32_t *slot = a.act_bits ? pl.slot : nullptr;      // act_bits implies need_slot
    // Few heads with long rows: a block per head would write for longer than a launch costs.  us, fill beside the selection /
    // spread over the chip, 8 heads, dh 64: 2048 rows (256 KB a head) 44.1 / 43.5, 4096 62.9 / 59.8, 16384 373 / 356; 64 heads
    // even.  The blocks of a caller's list have 256 threads instead of 1024: 1024 rows 25.9 / 23.6, 16384 119 / 57; 128 heads
    // of 2048 rows 39.7 / 35.9, 256 even.  With most rows active there is little to fill.
    const bool forced = a.forced_sel && a.U > 0;
    const int64_t head_bytes = (int64_t)a.L * a.dh * elem_size(dtype);
    const bool spread = !a.skip_fill && a.U * 2 <= a.L && BH < (forced ? 256 : 64) && head_bytes >= (forced ? 128 : 256) * 1024;
    auto fill_args = [&](auto *O, bool beside) {
        Fill<std::remove_pointer_t<decltype(O)>> f{};
        f.O = a.skip_fill || beside == spread ? nullptr : O; f.ldo = a.ldo; f.stats = pl.stats; f.head_group = a.head_group; f.hg_stride = a.hg_stride;
        f.pattern_id = a.pattern_id; f.nG = a.nG; f.dh = a.dh; f.row0 = a.row0; f.ext = a.ext;
        if (summed) { f.part = pl.score; f.parts = ceil_div(pl.Lp, 64); }
        return f;
    };
    const Fill<h16> fill16 = fill_args((h16 *)a.O, true);
    const Fill<float> fill32 = fill_args((float *)a.O, true);
    const bool v8 = a.ldo % 8 == 0 && ((uintptr_t)a.O % 16 == 0);              // 16-byte rows of O
    if (spread) {                                  // every row; the active pass writes its rows over it
        const int vec = dtype == SF_BF16 && v8 ? 8 : 4;
        const dim3 grid(ceil_div(a.L, 8 * (256 / (a.dh / vec))), BH);            // eight rows per thread
        if (dtype != SF_BF16) hipLaunchKernelGGL((fill_rows_kernel<4, float>), grid, dim3(256), 0, st, a.nH, a.L, fill_args((float *)a.O, false));
        else if (v8) hipLaunchKernelGGL((fill_rows_kernel<8, h16>), grid, dim3(256), 0, st, a.nH, a.L, fill_args((h16 *)a.O, false));
        else hipLaunchKernelGGL((fill_rows_kernel<4, h16>), grid, dim3(256), 0, st, a.nH, a.L, fill_args((h16 *)a.O, false));
    }
    const size_t key_bytes = (size_t)a.L * sizeof(uint32_t);
    if (forced) {
#define SF_FORCED_ARGS dim3(BH), dim3(256), key_bytes, st, a.forced_sel, userH, a.nH, a.L, a.U, sel, selH, slot, a.act_bits
        if (dtype != SF_BF16) hipLaunchKernelGGL((forced_slot_kernel<4, float>), SF_FORCED_ARGS, fill32);
        else if (v8) hipLaunchKernelGGL((forced_slot_kernel<8, h16>), SF_FORCED_ARGS, fill16);
        else hipLaunchKernelGGL((forced_slot_kernel<4, h16>), SF_FORCED_ARGS, fill16);
#undef SF_FORCED_ARGS
    } else {
        ScoreParts parts{nullptr, 0, 1, a.nH, nullptr, 0.f, nullptr, userH};
        if (a.U > 0 && a.U < a.L) {
            // the caller's score buffer takes the score itself: from the score kernel, or (parts) from the selection
            const bool direct = a.score_out && pl.score_parts == 1;
            const int scoreH = direct ? userH : a.nH;
            float *score = direct ? a.score_out : pl.score;
            // keys the score looks at: the sample's own keys, or the gathered key sample
            const void *Kx = a.K;
            sf_strides skx = a.sk;
            int Lk = a.L;
            const uint8_t *key_mask = a.key_valid;
            const float *kstats = pl.stats;
            const int32_t *nkeys = pl.n_valid;
            if (a.sample_idx && pl.Sp > 0) {
                const size_t gl = (size_t)ceil_div(a.L, 32) * 4 + (size_t)pl.Sp * 4;
                if (dtype == SF_BF16)
                    hipLaunchKernelGGL(gather_key_sample_kernel<h16>, dim3(BG), dim3(256), gl, st,
                                       (const h16 *)a.K, a.sk, a.key_valid, a.sample_idx, a.n_sample, a.nG, a.L,
                                       a.dh, pl.Sp, (h16 *)pl.ks, pl.ks_valid, pl.ks_stats, pl.n_keys, a.row0);
                else
                    hipLaunchKernelGGL(gather_key_sample_kernel<float>, dim3(BG), dim3(256), gl, st,
                                       (const float *)a.K, a.sk, a.key_valid, a.sample_idx, a.n_sample, a.nG, a.L,
                                       a.dh, pl.Sp, (float *)pl.ks, pl.ks_valid, pl.ks_stats, pl.n_keys, a.row0);
                Kx = pl.ks;
                skx.b = (int64_t)a.nG * pl.Sp * a.dh; skx.h = (int64_t)pl.Sp * a.dh; skx.l = a.dh;
                Lk = pl.Sp; key_mask = pl.ks_valid; kstats = pl.ks_stats; nkeys = pl.n_keys;
            }
            if (dtype == SF_BF16) {
                if (int32_t rc = score_bf16(a, Kx, skx, Lk, key_mask, kstats, score, scoreH, pl.score_parts, st)) return rc;
            } else {
                dim3 grid(ceil_div(a.L, SF32_TQ), BH);
                const size_t lds = (size_t)(SF32_TQ + SF32_TK) * (a.dh + 1) * sizeof(float);
                hipLaunchKernelGGL(score_f32_kernel, grid, dim3(256), lds, st, (const float *)a.Q, a.sq,
                                   (const float *)Kx, skx, a.head_group, a.hg_stride, a.pattern_id,
                                   a.key_valid, key_mask, nkeys, a.nH, a.L, Lk, a.dh, score, scoreH, a.row0,
                                   Kx == a.K);
            }
            parts = ScoreParts{score, (int64_t)a.B * scoreH * a.L, pl.score_parts, scoreH, nkeys,
                               1.0f / sqrtf((float)a.dh), pl.score_parts > 1 ? a.score_out : nullptr, userH};
        }
        // long rows, and rows of some length where there are few of them (6 rows of 512 scores: 7.9 us against 9.7 with 256),
        // get 1024 threads
        const bool wide = a.L >= 2048 || (a.L >= 512 && BH <= 256);
#define SF_SELECT_ARGS(NT) dim3(BH), dim3(NT), key_bytes, st, parts, a.key_valid, a.nH, a.L, a.U, a.u_active, sel, selH, slot, a.act_bits
#define SF_SELECT_LAUNCH(VEC, T, PART, F)                                                                        \
    do {                                                                                                         \
        if (wide) hipLaunchKernelGGL((select_kernel<1024, VEC, T, PART>), SF_SELECT_ARGS(1024), F);               \
        else hipLaunchKernelGGL((select_kernel<256, VEC, T, PART>), SF_SELECT_ARGS(256), F);                      \
    } while (0)
        if (dtype != SF_BF16) SF_SELECT_LAUNCH(4, float, false, fill32);
        else if (v8 && summed) SF_SELECT_LAUNCH(8, h16, true, fill16);
        else if (v8) SF_SELECT_LAUNCH(8, h16, false, fill16);
        else if (summed) SF_SELECT_LAUNCH(4, h16, true, fill16);
        else SF_SELECT_LAUNCH(4, h16, false, fill16);
#undef SF_SELECT_LAUNCH
#undef SF_SELECT_ARGS
    }

    // 3. active rows
    if (a.U > 0) {
        if (dtype == SF_BF16) {
            if (int32_t rc = attend_bf16(a, pl, Vuse, svu, sel, selH, st)) return rc;
        } else {
            dim3 grid(a.U, BH);
            hipLaunchKernelGGL(attend_f32_kernel, grid, dim3(64), a.L * sizeof(float), st, (const float *)a.Q,
                               a.sq, (const float *)a.K, a.sk, (const float *)Vuse, svu, v_sj, v_se,
                               a.head_group, a.hg_stride, a.pattern_id, a.key_valid, sel, selH, a.nH, a.L,
                               a.dh, a.U, (float *)a.O, a.ldo, a.row0);
        }
    }

    // 4. merge of the key splits
    if (pl.splits > 1) {
        const int64_t n_waves = (int64_t)BH * a.U;
        hipLaunchKernelGGL(merge_splits_kernel<h16>, dim3((unsigned)((n_waves + 3) / 4)), dim3(256), 0, st,
                           a.nH, a.L, a.dh, a.U, pl.Upad, pl.splits, n_waves, sel, selH, pl.part_o, pl.part_ml,
                           (h16 *)a.O, a.ldo, a.row0);
    }
    return check_launch("sparse_gqa_forward");
}

}  // namespace sf

using namespace sf;

static int32_t make_attn_args(const sf_desc *desc, int32_t nH, int32_t nG, Dims &D, AttnArgs &a)
{
    if (int32_t rc = read_desc(desc, D)) return rc;
    if (nH < 1 || nG < 1) return fail(SF_ERR_INVALID_ARG, "sparse_gqa: nH and nG must be positive");
    a = AttnArgs{};
    a.B = D.B; a.nH = nH; a.nG = nG; a.L = D.L; a.dh = D.dh; a.U = D.U; a.n_sample = D.n_sample;
    return SF_OK;
}

extern "C" size_t sf_sparse_gqa_workspace_bytes(const sf_desc *desc, int32_t nH, int32_t nG)
{
    Dims D; AttnArgs a;
    if (make_attn_args(desc, nH, nG, D, a)) return 0;
    a.v_transposed = 0;       // the larger of the two cases
    return attn_plan(D.dtype, a, nullptr).bytes;
}

extern "C" int32_t sf_sparse_gqa_plan(const sf_desc *desc, int32_t nH, int32_t nG, int32_t *plan_host)
{
    Dims D; AttnArgs a;
    if (int32_t rc = make_attn_args(desc, nH, nG, D, a)) return rc;
    if (!plan_host) return fail(SF_ERR_INVALID_ARG, "sparse_gqa_plan: NULL argument");
    if (D.dtype != SF_BF16) return fail(SF_ERR_UNSUPPORTED, "sparse_gqa_plan: 16-bit models only");
    const AttnPlan pl = attn_plan(D.dtype, a, nullptr);
    const bool whole = attend_short(a);
    plan_host[0] = pl.staged; plan_host[1] = pl.splits;
    plan_host[2] = whole ? 0 : pl.score_parts; plan_host[3] = whole ? 0 : pl.stat_parts;
    return SF_OK;
}

extern "C" int32_t sf_sparse_gqa_forward(const sf_desc *desc, int32_t nH, int32_t nG, const void *Q,
                                         sf_strides sq, const void *K, sf_strides sk, const void *V,
                                         sf_strides sv, int32_t v_transposed, const int32_t *head_group,
                                         const int32_t *pattern_id, const uint8_t *key_valid,
                                         const int32_t *sample_idx, const int32_t *forced_sel, void *O,
                                         int64_t ldo, int32_t *sel_out,
                                         float *score_out, void *workspace, size_t workspace_bytes,
                                         void *stream)
{
    Dims D; AttnArgs a;
    if (int32_t rc = make_attn_args(desc, nH, nG, D, a)) return rc;
    if (!Q || !K || !V || !head_group || !O) return fail(SF_ERR_INVALID_ARG, "sparse_gqa: NULL argument");
    if (ldo < (int64_t)nH * D.dh) return fail(SF_ERR_SHAPE, "sparse_gqa: ldo smaller than nH*dh");
    a.Q = Q; a.K = K; a.V = V; a.sq = sq; a.sk = sk; a.sv = sv; a.v_transposed = v_transposed != 0;
    a.head_group = head_group; a.hg_stride = nH; a.pattern_id = pattern_id; a.key_valid = key_valid;
    a.sample_idx = D.n_sample > 0 ? sample_idx : nullptr;
    a.forced_sel = forced_sel; a.O = O; a.ldo = ldo; a.sel_out = sel_out; a.score_out = score_out;
    a.ws = workspace; a.ws_bytes = workspace_bytes;
    return attention_forward(D.dtype, a, static_cast<hipStream_t>(stream));
}

// ---- sparse_gqa_forward for callers that cannot allocate --------------------------------------------------------
// The same launches as sf_sparse_gqa_forward with the workspace taken from a file-scope device array instead of a
// caller's buffer.  Every GPU the library runs on holds its own copy of the array at its own address until the
// process ends; the array's name is only a host-side handle, so its device address is looked up once per device
// (with that device current) and only that address is ever handed to a kernel.
static __device__ __align__(256) unsigned char scratch[SF_STATIC_SCRATCH_BYTES];

static int32_t static_scratch(void **out)
{
    constexpr int MAX_DEV = 64;
    static std::mutex mu;
    static void *per_device[MAX_DEV] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEV)
        return fail(SF_ERR_HIP, "sparse_gqa_static: no current device (or device index >= %d)", MAX_DEV);
    std::lock_guard<std::mutex> lock(mu);
    if (!per_device[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(SF_ERR_HIP, "sparse_gqa_static: hipGetSymbolAddress failed on device %d: %s", dev,
                        hipGetErrorString(e));
        per_device[dev] = p;
    }
    *out = per_device[dev];
    return SF_OK;
}

extern "C" size_t sf_sparse_gqa_static_capacity(void) { return SF_STATIC_SCRATCH_BYTES; }

extern "C" int32_t sf_sparse_gqa_forward_static(const sf_desc *desc, int32_t nH, int32_t nG, const void *Q,
                                                sf_strides sq, const void *K, sf_strides sk, const void *V,
                                                sf_strides sv, int32_t v_transposed, const int32_t *head_group,
                                                const int32_t *pattern_id, const uint8_t *key_valid,
                                                const int32_t *sample_idx, const int32_t *forced_sel, void *O,
                                                int64_t ldo, int32_t *sel_out, float *score_out, void *stream)
{
    Dims D; AttnArgs a;
    if (int32_t rc = make_attn_args(desc, nH, nG, D, a)) return rc;
    a.v_transposed = v_transposed != 0;
    a.ws_bytes = SF_STATIC_SCRATCH_BYTES;
    const size_t need = attn_plan(D.dtype, a, nullptr).bytes;
    if (need > SF_STATIC_SCRATCH_BYTES)
        return fail(SF_ERR_WORKSPACE,
                    "sparse_gqa_static: this problem needs %zu bytes of scratch, the built-in buffer holds %zu; use "
                    "sf_sparse_gqa_forward with a workspace of sf_sparse_gqa_workspace_bytes()",
                    need, (size_t)SF_STATIC_SCRATCH_BYTES);
    void *ws = nullptr;
    if (int32_t rc = static_scratch(&ws)) return rc;
    // Nothing in the buffer has to start at zero: every piece (transposed V, K/V statistics, scores, active lists,
    // row -> slot map, key-split partials) is written in full by an earlier kernel of the same call before a later
    // one reads it, exactly as with a caller's uninitialised workspace.
    return sf_sparse_gqa_forward(desc, nH, nG, Q, sq, K, sk, V, sv, v_transposed, head_group, pattern_id, key_valid,
                                 sample_idx, forced_sel, O, ldo, sel_out, score_out, ws, SF_STATIC_SCRATCH_BYTES, stream);
}
