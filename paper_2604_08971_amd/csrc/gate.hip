// SentryGate on the device: the importance scores of Eq. (1) for every layer and presence pattern, and
// the global threshold that meets a cost budget (Sec. 4.5, the paragraph that introduces the three pruning
// locations; Sec. 4.2 names the FLOPs / energy budget).  Both are plan-construction steps: tiny next to the
// encoder forward, so the kernels aim at being exact and launch-cheap, not at a roofline.
#include <atomic>
#include <type_traits>

#include "common.hpp"
#include "topk.hpp"

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
// as a weighted selection: v, the largest key at which the cost exceeds the budget; the keep set is { key > v }.  One
// histogram of costs over 1024 equal steps of the score's range finds the step that holds v, and its few units are summed
// up pair by pair; where it has more than 64 of them, a sample of the channels shows many in one step, or the scores are no
// finite range, a radix select (eight bits per pass over a histogram of costs) finds v.  Costs are integers: the order of the
// atomics does not matter.
//
// One block and latency-bound: the scores are read once, eight loads of a thread in flight, and kept in LDS where they
// fit; layers are shared by all waves.  us a call, the radix passes alone with loads one after the other and a wave per layer /
// this: 6 layers of 8 heads and 2048 channels 38 / 18.5, their scores all equal 52 / 34, two values 42 / 39, nine zeros in
// ten 54 / 39, an outlier 38 / 37; 64 layers of 64 heads, groups and 512 channels 156 / 67.
constexpr int BUDGET_NT = 1024, BUDGET_BINS = 1024, BUDGET_LIST = 64;
constexpr int BUDGET_LDS_KEYS = 38000;                                // keys in LDS (152 KB)

__global__ __launch_bounds__(BUDGET_NT) void budget_search_kernel(
    const float *__restrict__ gh, const float *__restrict__ gf, int64_t lstride_h, int64_t lstride_f, int nl, int Hq,
    int Hk, int F, uint32_t f_magic, int cached, int cached_h, BudgetCosts costs, int64_t c_fixed, int64_t budget, float *__restrict__ tau_out,
    int32_t *__restrict__ k_head_out, int32_t *__restrict__ k_ffn_out, int64_t *__restrict__ cost_out,
    int32_t *__restrict__ feasible_out)
{
    extern __shared__ uint32_t gkey[];                                // [nl][Hk] largest key of a group's heads, [nl][Hq] when cached_h, [nl][F] when cached
    __shared__ unsigned long long hist[BUDGET_BINS];
    __shared__ unsigned long long best64[MAX_LAYERS_BUDGET];          // key and complement of the index: first of the largest channels
    __shared__ int best_h[MAX_LAYERS_BUDGET], best_g[MAX_LAYERS_BUDGET], best_f[MAX_LAYERS_BUDGET], n_f[MAX_LAYERS_BUDGET];
    __shared__ long long list_cost[BUDGET_LIST];
    __shared__ uint32_t list_key[BUDGET_LIST];
    __shared__ uint32_t s_max, s_low, s_min, s_digit;
    __shared__ long long s_rest, s_cost;
    __shared__ int s_found, s_many, s_list;
    uint32_t *hkeys = gkey + nl * Hk, *fkeys = hkeys + (cached_h ? nl * Hq : 0);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int NWAVES = BUDGET_NT / 64;
    // the channels of a layer are shared by `parts` waves: share w of nl * parts
    const int parts = nl < NWAVES ? NWAVES / nl : 1;

    auto key_h = [&](int l, int i) { return cached_h ? hkeys[l * Hq + i] : score_key(gh[l * lstride_h + i]); };
    auto key_f = [&](int l, int i) { return cached ? fkeys[l * F + i] : score_key(gf[l * lstride_f + i]); };

    if (tid == 0) { s_max = 0u; s_low = s_min = 0xffffffffu; s_cost = 0; s_list = 0; }
    for (int j = tid; j < BUDGET_BINS; j += BUDGET_NT) hist[j] = 0ull;
    for (int l = tid; l < nl; l += BUDGET_NT) { best64[l] = 0ull; n_f[l] = 0; }
    if (cached_h)
        for (int t = tid; t < nl * Hq; t += BUDGET_NT) hkeys[t] = score_key(gh[t / Hq * lstride_h + t % Hq]);
    if (cached) {
        constexpr int UN = 8;
        for (int t0 = 0; t0 < nl * F; t0 += UN * BUDGET_NT) {
            float v[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int t = t0 + u * BUDGET_NT + tid, l = F > 1 ? (int)__umulhi((uint32_t)t, f_magic) : t;      // t / F
                v[u] = t < nl * F ? gf[l * lstride_f + (t - l * F)] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int t = t0 + u * BUDGET_NT + tid;
                if (t < nl * F) fkeys[t] = score_key(v[u]);
            }
        }
    }
    __syncthreads();

    // the best head, group and channel of a layer (first of the largest), the groups' keys, the range of all keys
    for (int w = wave; w < nl * parts; w += NWAVES) {
        const int l = w / parts;
        uint32_t mk = 0u, lo = 0xffffffffu;
        int mi = -1;
#pragma unroll 4
        for (int i = w % parts * 64 + lane; i < F; i += parts * 64) {
            const uint32_t k = key_f(l, i);
            lo = min(lo, k);
            if (k > mk || mi < 0) { mk = k; mi = i; }
        }
        const uint32_t m = wave_max_u32(mk), at = wave_max_u32(mi >= 0 && mk == m ? ~(uint32_t)mi : 0u);
        lo = ~wave_max_u32(~lo);
        if (lane == 0 && at) {                                        // at 0: no channel in this share
            atomicMax(&best64[l], (unsigned long long)m << 32 | at);
            atomicMax(&s_max, m);
            atomicMin(&s_low, lo);
        }
    }
    const int per_group = Hq / Hk;
    for (int l = wave; l < nl; l += NWAVES) {
        uint32_t mk = 0u, lo = 0xffffffffu;
        int mi = -1;
        for (int i = lane; i < Hq; i += 64) {
            const uint32_t k = key_h(l, i);
            lo = min(lo, k);
            if (k > mk || mi < 0) { mk = k; mi = i; }
        }
        const uint32_t m = wave_max_u32(mk), at = wave_max_u32(mi >= 0 && mk == m ? ~(uint32_t)mi : 0u);
        lo = ~wave_max_u32(~lo);
        if (lane == 0) {
            best_h[l] = (int)~at;
            best_g[l] = (int)~at / per_group;                         // the best head's group
            atomicMax(&s_max, m);
            atomicMin(&s_low, lo);
        }
        if (lane < Hk) {
            uint32_t g = 0u;
            for (int j = 0; j < per_group; ++j) g = max(g, key_h(l, lane * per_group + j));
            gkey[l * Hk + lane] = g;
        }
    }
    __syncthreads();
    for (int l = tid; l < nl; l += BUDGET_NT) best_f[l] = (int)~(uint32_t)best64[l];
    __syncthreads();

    // every unit but the ones that always stay: visit(key, in, cost)
    auto units = [&](auto visit) {
        for (int l = 0; l < nl; ++l) {
            const int bf = best_f[l];
            const int64_t cost = costs.ffn[l];
            for (int i0 = 0; i0 < F; i0 += BUDGET_NT) {
                const int i = i0 + tid;
                const bool in = i < F && i != bf;
                visit(in ? key_f(l, i) : 0u, in, cost);
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
            visit(in ? gkey[t] : 0u, in, in ? costs.group[l] : 0);
        }
    };
    long long base = c_fixed;
    for (int l = 0; l < nl; ++l) base += costs.head[l] + costs.group[l] + costs.ffn[l];

    // A unit in the histogram of a radix pass.  Atomics on one address run one after the other: where many scores meet in a bin
    // (`crowded`), lanes with the bin and the cost of the first one are added by it, twice; the others by themselves.
    bool crowded = true;
    auto add = [&](bool use, int bin, int64_t cost) {
        if (crowded)
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const unsigned long long left = __ballot(use);
                if (!left) return;
                const int src = __ffsll((long long)left) - 1;
                const int b = __builtin_amdgcn_readlane(bin, src);
                const int64_t c = (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(cost >> 32), src) << 32 |
                                            (uint32_t)__builtin_amdgcn_readlane((int)cost, src));
                const unsigned long long same = __ballot(use && bin == b && cost == c);
                if (lane == src) atomicAdd(&hist[b], (unsigned long long)c * (unsigned long long)__popcll(same));
                use = use && !(bin == b && cost == c);
            }
        if (use) atomicAdd(&hist[bin], (unsigned long long)cost);
    };
    // a wave's lane owns PER consecutive bins of a histogram: the bin in which the cost from the top passes `rest`
    auto scan = [&](auto per, long long rest) {
        constexpr int PER = decltype(per)::value;
        long long h[PER], local = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) { h[j] = (long long)hist[PER * lane + j]; local += h[j]; }
        long long incl = local;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const long long t = __shfl_down(incl, o);
            if (lane + o < 64) incl += t;
        }
        long long run = incl - local;                                 // cost of the strictly higher bins
#pragma unroll
        for (int j = PER - 1; j >= 0; --j) {
            if (run <= rest && run + h[j] > rest) { s_digit = (uint32_t)(PER * lane + j); s_cost = rest - run; s_found = 1; }
            run += h[j];
        }
    };
    uint32_t v = 0u;
    bool exceeds = budget >= base;                                    // is there a key at which the budget is exceeded?
    bool open = exceeds;                                              // v still to be found
    const float vlo = key_score(s_low);
    float per_unit;
    bool steps = open && cut_range(vlo, key_score(s_max), BUDGET_BINS, per_unit);
    auto bin_of = [&](uint32_t key) { return step_of(key_score(key), vlo, per_unit, BUDGET_BINS); };
    if (steps) {
        // a channel per thread, spread over the layers: where a quarter of a wave's meet in a step, the others do, in this histogram
        // and in the list of a step
        const int t = tid * max(1, nl * F / BUDGET_NT), bin = t < nl * F ? bin_of(key_f(t / F, t % F)) : -1;
        if (tid == 0) { s_found = 0; s_many = 0; }
        __syncthreads();
        const int first = __builtin_amdgcn_readfirstlane(bin);
        if (first >= 0 && __popcll(__ballot(bin == first)) > 16) s_many = 1;
        __syncthreads();
        crowded = s_many;
        steps = !crowded;
    }
    if (steps) {
        units([&](uint32_t key, bool in, int64_t cost) {
            if (in) atomicAdd(&hist[bin_of(key)], (unsigned long long)cost);
        });
        __syncthreads();
        if (tid < 64) scan(std::integral_constant<int, BUDGET_BINS / 64>(), budget - base);
        __syncthreads();
        if (!s_found) {                                               // everything fits
            exceeds = open = false;
        } else {
            const int bin = (int)s_digit;
            const long long rest = s_cost;
            units([&](uint32_t key, bool in, int64_t cost) {
                if (in && bin_of(key) == bin) {
                    const int at = atomicAdd(&s_list, 1);
                    if (at < BUDGET_LIST) { list_key[at] = key; list_cost[at] = cost; }
                }
            });
            __syncthreads();
            const int n = s_list;
            if (n <= BUDGET_LIST) {
                const uint32_t mine = lane < n ? list_key[lane] : 0u;
                long long sum = 0;                                    // cost of the step's units with this key or a larger one
                for (int j = 0; j < n; ++j) sum += list_key[j] >= mine ? list_cost[j] : 0;
                v = wave_max_u32(lane < n && sum > rest ? mine : 0u);
                open = false;
            }
        }
        __syncthreads();
    }
    if (open) {
        uint32_t mask = 0u;
        if (tid == 0) s_rest = budget - base;
        for (int pass = 0; pass < 4; ++pass) {                        // uniform over the block
            const int shift = 24 - 8 * pass;
            for (int j = tid; j < 256; j += BUDGET_NT) hist[j] = 0ull;
            if (tid == 0) s_found = 0;
            __syncthreads();
            units([&](uint32_t key, bool in, int64_t cost) {
                add(in && (key & mask) == v, (int)((key >> shift) & 255u), cost);
            });
            __syncthreads();
            if (tid < 64) scan(std::integral_constant<int, 4>(), s_rest);
            __syncthreads();
            if (!s_found) { exceeds = false; break; }                 // pass 0 only: everything fits
            v |= s_digit << shift;
            mask |= 255u << shift;
            if (tid == 0) s_rest = s_cost;
            __syncthreads();
        }
    }
    // v: the largest key at which the budget is exceeded.  The strictest threshold is the largest score itself.
    const bool feasible = budget >= base && !(exceeds && v >= s_max);
    const uint32_t lo = exceeds ? v + 1u : 0u;                        // keep { key >= lo }; unused when infeasible
    __syncthreads();
    if (tid == 0) s_cost = 0;
    if (feasible)
        for (int w = wave; w < nl * parts; w += NWAVES) {
            const int l = w / parts;
            int kf = 0;
            uint32_t mk = 0xffffffffu;
#pragma unroll 4
            for (int i = w % parts * 64 + lane; i < F; i += parts * 64) {
                const uint32_t k = key_f(l, i);
                if (k >= lo) { ++kf; mk = min(mk, k); }
            }
            kf = wave_incl_scan(kf);
            mk = ~wave_max_u32(~mk);
            if (lane == 63) {
                atomicAdd(&n_f[l], kf);
                atomicMin(&s_min, mk);
            }
        }
    __syncthreads();
    for (int l = wave; l < nl; l += NWAVES) {
        int kh = 0, kg = 0;
        uint32_t mk = 0xffffffffu;
        if (feasible) {
            for (int i = lane; i < Hq; i += 64) {
                const uint32_t k = key_h(l, i);
                if (k >= lo) { ++kh; mk = min(mk, k); }
            }
            if (lane < Hk) kg = gkey[l * Hk + lane] >= lo;
        }
        kh = wave_incl_scan(kh);
        kg = wave_incl_scan(kg);
        mk = ~wave_max_u32(~mk);
        if (lane == 63) {
            if (kh == 0) { kh = 1; kg = 1; }                          // the best head stays, with its group
            const int kf = max(n_f[l], 1);                            // the best channel stays
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
    int64_t keys = (int64_t)D.nl * D.Hk;                              // the groups' always; the channels', then the heads' where they fit
    const bool cached = keys + (int64_t)D.nl * D.F <= BUDGET_LDS_KEYS;
    if (cached) keys += (int64_t)D.nl * D.F;
    const bool cached_h = keys + (int64_t)D.nl * D.Hq <= BUDGET_LDS_KEYS;
    if (cached_h) keys += (int64_t)D.nl * D.Hq;
    const size_t lds = (size_t)keys * sizeof(uint32_t);
    const uint32_t f_magic = (uint32_t)((((uint64_t)1 << 32) + D.F - 1) / D.F);      // t / F = umulhi(t, f_magic) for t F < 2^32
    static std::atomic<bool> attr_set{false};     // setting the attribute twice is harmless
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(budget_search_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, BUDGET_LDS_KEYS * 4) != hipSuccess)
            return fail(SF_ERR_HIP, "budget_search: cannot reserve %d bytes of LDS", BUDGET_LDS_KEYS * 4);
        attr_set = true;
    }
    hipLaunchKernelGGL(budget_search_kernel, dim3(1), dim3(BUDGET_NT), lds, static_cast<hipStream_t>(stream),
                       g_head + (int64_t)pattern * D.Hq, g_ffn + (int64_t)pattern * D.F, (int64_t)D.P * D.Hq,
                       (int64_t)D.P * D.F, D.nl, D.Hq, D.Hk, D.F, f_magic, cached, cached_h, bc, c_fixed, budget, tau, k_head, k_ffn, cost, feasible);
    return check_launch("budget_search");
}
