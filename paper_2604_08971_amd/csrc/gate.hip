// SentryGate on the device: the importance scores of Eq. (1) for every layer and presence pattern, and
// the global threshold that meets a cost budget (Sec. 4.5, the paragraph that introduces the three pruning
// locations; Sec. 4.2 names the FLOPs / energy budget).  Both are plan-construction steps: tiny next to the
// encoder forward, so the kernels aim at being exact and launch-cheap, not at a roofline.
#include <atomic>

#include "common.hpp"

namespace sf {

namespace {

constexpr int MAX_HIDDEN = 1024;
constexpr int MAX_LAYERS_BUDGET = 64;

// g[l, p, i] = sigmoid(zeta[l, i] + gamma[l] * (Wb[l, i, :] . h + cb[l, i])),  h = nonlin(Wa[l] m_p + ba[l]).
// grid (ceil(n_units / 256), P, nl).  Eight lanes share one unit's output row (one 128-byte line per step).
__global__ __launch_bounds__(256) void gate_eval_kernel(
    const float *__restrict__ Wa, const float *__restrict__ ba, const float *__restrict__ Wb,
    const float *__restrict__ cb, const float *__restrict__ zeta, const float *__restrict__ gamma,
    const int32_t *__restrict__ pattern_bits, int M, int Hd, int n_units, int Hq, int nonlin, int P,
    float *__restrict__ g_head, float *__restrict__ g_ffn)
{
    __shared__ float h[MAX_HIDDEN];
    const int l = blockIdx.z, p = blockIdx.y;
    const uint32_t bits = (uint32_t)pattern_bits[p];
    for (int r = threadIdx.x; r < Hd; r += 256) {
        float a = ba ? ba[(int64_t)l * Hd + r] : 0.f;
        for (int j = 0; j < M; ++j)
            if ((bits >> j) & 1u) a += Wa[((int64_t)l * Hd + r) * M + j];
        h[r] = nonlin == 0 ? fmaxf(a, 0.f) : tanhf(a);
    }
    __syncthreads();
    const int sub = threadIdx.x & 7;
    const int F = n_units - Hq;
    const float gm = gamma[l];
    for (int u0 = 0; u0 < 256; u0 += 32) {
        const int i = blockIdx.x * 256 + u0 + (threadIdx.x >> 3);       // uniform over the 8 lanes of a unit
        float acc = 0.f;
        if (i < n_units) {
            const float *w = Wb + ((int64_t)l * n_units + i) * Hd;
            if ((Hd & 3) == 0) {
                for (int r = sub * 4; r < Hd; r += 32) {
                    const f32x4 q = *reinterpret_cast<const f32x4 *>(w + r);
                    acc = fmaf(q[0], h[r], acc);
                    acc = fmaf(q[1], h[r + 1], acc);
                    acc = fmaf(q[2], h[r + 2], acc);
                    acc = fmaf(q[3], h[r + 3], acc);
                }
            } else {
                for (int r = sub; r < Hd; r += 8) acc = fmaf(w[r], h[r], acc);
            }
        }
        acc += __shfl_xor(acc, 1);
        acc += __shfl_xor(acc, 2);
        acc += __shfl_xor(acc, 4);
        if (i < n_units && sub == 0) {
            const float f = acc + (cb ? cb[(int64_t)l * n_units + i] : 0.f);
            const float z = zeta[(int64_t)l * n_units + i] + gm * f;
            const float g = 1.f / (1.f + expf(-z));
            if (i < Hq) g_head[((int64_t)l * P + p) * Hq + i] = g;
            else g_ffn[((int64_t)l * P + p) * F + (i - Hq)] = g;
        }
    }
}

// Order-preserving map float -> uint32 (a >= b  <=>  key(a) >= key(b) for non-NaN; -0 and +0 share a key)
__device__ inline uint32_t score_key(float f)
{
    if (f == 0.f) f = 0.f;
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float key_score(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

struct BudgetCosts { int64_t head[MAX_LAYERS_BUDGET], group[MAX_LAYERS_BUDGET], ffn[MAX_LAYERS_BUDGET]; };

// The cost of a threshold K is a weighted count: c_fixed, plus one head, one K/V group and one channel per layer (which
// always stay), plus the cost of every other unit whose key is >= K - heads and channels with their own keys, a K/V
// group with the largest key of its heads, one best unit of each kind and layer left out.  So the threshold is found
// as a weighted radix select: v, the largest key at which the cost exceeds the budget, eight bits per pass over a
// histogram of costs (integers: the order of the atomics does not matter); the keep set is { key > v }.
//
// One block and latency-bound: the scores are read once (into LDS where they fit) and passed over four times, where a
// bisection over the key's bits takes 32 passes.  Six layers of 8 heads and 2048 channels: 260 -> 16 us.
constexpr int BUDGET_NT = 1024;
constexpr int BUDGET_LDS_KEYS = 32768;                                // channels cached in LDS (128 KB)

__global__ __launch_bounds__(BUDGET_NT) void budget_search_kernel(
    const float *__restrict__ gh, const float *__restrict__ gf, int64_t lstride_h, int64_t lstride_f, int nl, int Hq,
    int Hk, int F, int cached, BudgetCosts costs, int64_t c_fixed, int64_t budget, float *__restrict__ tau_out,
    int32_t *__restrict__ k_head_out, int32_t *__restrict__ k_ffn_out, int64_t *__restrict__ cost_out,
    int32_t *__restrict__ feasible_out)
{
    extern __shared__ uint32_t fkeys[];                               // [nl][F] when cached
    __shared__ unsigned long long hist[256];
    __shared__ uint32_t gkey[MAX_LAYERS_BUDGET * 64];                 // [nl][Hk] largest key of a group's heads
    __shared__ int best_h[MAX_LAYERS_BUDGET], best_g[MAX_LAYERS_BUDGET], best_f[MAX_LAYERS_BUDGET];
    __shared__ uint32_t s_max, s_min, s_digit;
    __shared__ long long s_rest, s_cost;
    __shared__ int s_found;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int NWAVES = BUDGET_NT / 64;

    auto key_h = [&](int l, int i) { return score_key(gh[l * lstride_h + i]); };
    auto key_f = [&](int l, int i) { return cached ? fkeys[l * F + i] : score_key(gf[l * lstride_f + i]); };

    if (tid == 0) { s_max = 0u; s_min = 0xffffffffu; s_cost = 0; }
    if (cached)
        for (int l = 0; l < nl; ++l)
            for (int i = tid; i < F; i += BUDGET_NT) fkeys[l * F + i] = score_key(gf[l * lstride_f + i]);
    __syncthreads();

    // a wave per layer: the best head, group and channel (first of the largest) and the groups' keys
    auto first_of_max = [&](uint32_t mk, int mi, int &idx) {          // over the wave
        uint32_t m = mk;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o));
        int at = mk == m ? mi : 0x7fffffff;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) at = min(at, __shfl_xor(at, o));
        idx = at;
        return m;
    };
    const int per_group = Hq / Hk;
    for (int l = wave; l < nl; l += NWAVES) {
        uint32_t mk = 0u;
        int mi = 0x7fffffff, idx;
        for (int i = lane; i < F; i += 64) {
            const uint32_t k = key_f(l, i);
            if (k > mk || mi == 0x7fffffff) { mk = k; mi = i; }
        }
        const uint32_t mf = first_of_max(mk, mi, idx);
        if (lane == 0) best_f[l] = idx;
        mk = 0u;
        mi = 0x7fffffff;
        for (int i = lane; i < Hq; i += 64) {
            const uint32_t k = key_h(l, i);
            if (k > mk || mi == 0x7fffffff) { mk = k; mi = i; }
        }
        const uint32_t mh = first_of_max(mk, mi, idx);
        if (lane == 0) {
            best_h[l] = idx;
            best_g[l] = idx / per_group;                              // the best head's group
            atomicMax(&s_max, max(mf, mh));
        }
        if (lane < Hk) {
            uint32_t g = 0u;
            for (int j = 0; j < per_group; ++j) g = max(g, key_h(l, lane * per_group + j));
            gkey[l * 64 + lane] = g;
        }
    }
    __syncthreads();

    // every unit but the ones that always stay: visit(key, cost, everyone in the wave has the same cost)
    auto units = [&](auto visit) {
        for (int l = 0; l < nl; ++l) {
            const int bf = best_f[l];
            for (int i0 = 0; i0 < F; i0 += BUDGET_NT) {
                const int i = i0 + tid;
                const bool in = i < F && i != bf;
                visit(in ? key_f(l, i) : 0u, in, costs.ffn[l]);
            }
        }
        for (int t0 = 0; t0 < nl * Hq; t0 += BUDGET_NT) {
            const int t = t0 + tid, l = t / Hq, i = t % Hq;
            const bool in = t < nl * Hq && i != best_h[l];
            visit(in ? key_h(l, i) : 0u, in, in ? costs.head[l] : 0);
        }
        for (int t0 = 0; t0 < nl * Hk; t0 += BUDGET_NT) {
            const int t = t0 + tid, l = t / Hk, i = t % Hk;
            const bool in = t < nl * Hk && i != best_g[l];
            visit(in ? gkey[l * 64 + i] : 0u, in, in ? costs.group[l] : 0);
        }
    };
    long long base = c_fixed;
    for (int l = 0; l < nl; ++l) base += costs.head[l] + costs.group[l] + costs.ffn[l];

    uint32_t v = 0u, mask = 0u;
    bool exceeds = budget >= base;                                    // is there a key at which the budget is exceeded?
    if (tid == 0) s_rest = budget - base;
    if (exceeds)
        for (int pass = 0; pass < 4; ++pass) {                        // uniform over the block
            const int shift = 24 - 8 * pass;
            for (int j = tid; j < 256; j += BUDGET_NT) hist[j] = 0ull;
            if (tid == 0) s_found = 0;
            __syncthreads();
            units([&](uint32_t key, bool in, int64_t cost) {
                const bool use = in && (key & mask) == v;
                const uint32_t bin = (key >> shift) & 255u;
                if (pass == 0) {
                    // scores of one layer share a few exponents: one atomic per wave, bin and cost
                    unsigned long long left = __ballot(use);
                    while (left) {
                        const int src = __ffsll((long long)left) - 1;
                        const uint32_t b = (uint32_t)__shfl((int)bin, src);
                        const long long c = __shfl((long long)cost, src);
                        const unsigned long long same = __ballot(use && bin == b && cost == c) & left;
                        if (lane == src) atomicAdd(&hist[b], (unsigned long long)c * (unsigned long long)__popcll(same));
                        left &= ~same;
                    }
                } else if (use) {
                    atomicAdd(&hist[bin], (unsigned long long)cost);
                }
            });
            __syncthreads();
            if (tid < 64) {
                // lane owns bins 4*lane .. 4*lane+3: the bin in which the cost from the top passes the rest of the budget
                long long h[4], local = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) { h[j] = (long long)hist[4 * lane + j]; local += h[j]; }
                long long incl = local;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const long long t = __shfl_down(incl, o);
                    if (lane + o < 64) incl += t;
                }
                const long long rest = s_rest;
                long long run = incl - local;                         // cost of the strictly higher bins
#pragma unroll
                for (int j = 3; j >= 0; --j) {
                    if (run <= rest && run + h[j] > rest) { s_digit = (uint32_t)(4 * lane + j); s_cost = rest - run; s_found = 1; }
                    run += h[j];
                }
            }
            __syncthreads();
            if (!s_found) { exceeds = false; break; }                 // pass 0 only: everything fits
            v |= s_digit << shift;
            mask |= 255u << shift;
            if (tid == 0) s_rest = s_cost;
            __syncthreads();
        }
    // v: the largest key at which the budget is exceeded.  The strictest threshold is the largest score itself.
    const bool feasible = budget >= base && !(exceeds && v >= s_max);
    const uint32_t lo = exceeds ? v + 1u : 0u;                        // keep { key >= lo }; unused when infeasible
    __syncthreads();
    if (tid == 0) s_cost = 0;
    __syncthreads();
    for (int l = wave; l < nl; l += NWAVES) {
        int kf = 0, kh = 0, kg = 0;
        uint32_t mk = 0xffffffffu;
        if (feasible) {
            for (int i = lane; i < F; i += 64) {
                const uint32_t k = key_f(l, i);
                if (k >= lo) { ++kf; mk = min(mk, k); }
            }
            for (int i = lane; i < Hq; i += 64) {
                const uint32_t k = key_h(l, i);
                if (k >= lo) { ++kh; mk = min(mk, k); }
            }
            if (lane < Hk) kg = gkey[l * 64 + lane] >= lo;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            kf += __shfl_xor(kf, o);
            kh += __shfl_xor(kh, o);
            kg += __shfl_xor(kg, o);
            mk = min(mk, (uint32_t)__shfl_xor((int)mk, o));
        }
        if (lane == 0) {
            if (kh == 0) { kh = 1; kg = 1; }                          // the best head stays, with its group
            if (kf == 0) kf = 1;                                      // the best channel stays
            k_head_out[l] = kh;
            k_ffn_out[l] = kf;
            atomicAdd(reinterpret_cast<unsigned long long *>(&s_cost),
                      (unsigned long long)(kh * costs.head[l] + kg * costs.group[l] + kf * costs.ffn[l]));
            atomicMin(&s_min, mk);
        }
    }
    __syncthreads();
    if (tid == 0) {
        *tau_out = feasible ? key_score(s_min) : INFINITY;            // the smallest score that is kept
        *cost_out = c_fixed + s_cost;
        *feasible_out = feasible ? 1 : 0;
    }
}

}  // namespace

}  // namespace sf

using namespace sf;

extern "C" int32_t sf_gate_eval(const sf_desc *desc, const sf_gate_params *gp, const int32_t *pattern_bits,
                                float *g_head, float *g_ffn, void *stream)
{
    Dims D;
    if (int32_t rc = read_desc(desc, D)) return rc;
    if (!gp || !pattern_bits || !g_head || !g_ffn) return fail(SF_ERR_INVALID_ARG, "gate_eval: NULL argument");
    if (gp->n_modalities < 1 || gp->n_modalities > 32 || gp->hidden < 1 || gp->hidden > MAX_HIDDEN)
        return fail(SF_ERR_INVALID_ARG, "gate_eval: needs 1 <= n_modalities <= 32 and 1 <= hidden <= %d", MAX_HIDDEN);
    if (gp->nonlin != SF_GATE_RELU && gp->nonlin != SF_GATE_TANH)
        return fail(SF_ERR_UNSUPPORTED, "gate_eval: unknown nonlinearity");
    if (!gp->Wa || !gp->Wb || !gp->zeta || !gp->gamma) return fail(SF_ERR_INVALID_ARG, "gate_eval: NULL parameter pointer");
    if ((uintptr_t)gp->Wb & 15) return fail(SF_ERR_INVALID_ARG, "gate_eval: Wb must be 16-byte aligned");
    if (D.P > 65535 || D.nl > 65535) return fail(SF_ERR_SHAPE, "gate_eval: too many patterns or layers");
    const int n_units = D.Hq + D.F;
    dim3 grid(ceil_div(n_units, 256), D.P, D.nl);
    hipLaunchKernelGGL(gate_eval_kernel, grid, dim3(256), 0, static_cast<hipStream_t>(stream), (const float *)gp->Wa,
                       (const float *)gp->ba, (const float *)gp->Wb, (const float *)gp->cb, (const float *)gp->zeta,
                       (const float *)gp->gamma, pattern_bits, gp->n_modalities, gp->hidden, n_units, D.Hq, gp->nonlin,
                       D.P, g_head, g_ffn);
    return check_launch("gate_eval");
}

extern "C" int32_t sf_budget_search(const sf_desc *desc, const float *g_head, const float *g_ffn, int32_t pattern,
                                    const int64_t *c_head_host, const int64_t *c_group_host,
                                    const int64_t *c_ffn_host, int64_t c_fixed, int64_t budget, float *tau,
                                    int32_t *k_head, int32_t *k_ffn, int64_t *cost, int32_t *feasible, void *stream)
{
    Dims D;
    if (int32_t rc = read_desc(desc, D)) return rc;
    if (!g_head || !g_ffn || !c_head_host || !c_group_host || !c_ffn_host || !tau || !k_head || !k_ffn || !cost ||
        !feasible)
        return fail(SF_ERR_INVALID_ARG, "budget_search: NULL argument");
    if (pattern < 0 || pattern >= D.P) return fail(SF_ERR_INVALID_ARG, "budget_search: pattern %d out of range", pattern);
    if (D.nl > MAX_LAYERS_BUDGET) return fail(SF_ERR_SHAPE, "budget_search: at most %d layers", MAX_LAYERS_BUDGET);
    if (D.Hk > 64) return fail(SF_ERR_SHAPE, "budget_search: at most 64 K/V groups");
    BudgetCosts bc{};
    for (int l = 0; l < D.nl; ++l) {
        if (c_head_host[l] < 0 || c_group_host[l] < 0 || c_ffn_host[l] < 0)
            return fail(SF_ERR_INVALID_ARG, "budget_search: negative cost in layer %d", l);
        bc.head[l] = c_head_host[l]; bc.group[l] = c_group_host[l]; bc.ffn[l] = c_ffn_host[l];
    }
    const bool cached = (int64_t)D.nl * D.F <= BUDGET_LDS_KEYS;
    const size_t lds = cached ? (size_t)D.nl * D.F * sizeof(uint32_t) : 0;
    static std::atomic<bool> attr_set{false};     // setting the attribute twice is harmless
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(budget_search_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, BUDGET_LDS_KEYS * 4) != hipSuccess)
            return fail(SF_ERR_HIP, "budget_search: cannot reserve %d bytes of LDS", BUDGET_LDS_KEYS * 4);
        attr_set = true;
    }
    hipLaunchKernelGGL(budget_search_kernel, dim3(1), dim3(BUDGET_NT), lds, static_cast<hipStream_t>(stream),
                       g_head + (int64_t)pattern * D.Hq, g_ffn + (int64_t)pattern * D.F, (int64_t)D.P * D.Hq,
                       (int64_t)D.P * D.F, D.nl, D.Hq, D.Hk, D.F, cached ? 1 : 0, bc, c_fixed, budget, tau, k_head, k_ffn, cost, feasible);
    return check_launch("budget_search");
}
