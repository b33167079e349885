// SentryAttend on bf16 MFMA (Sec. 4.4 of the paper, Eq. (6)).
//
// Both kernels compute the TRANSPOSED score tile S^T = K_tile . Q^T with
// 32x32x16 MFMAs, so that one accumulator lane owns ONE query (column
// lane % 32) and 16 of the tile's 32 keys.  Everything the softmax needs per
// query (running max, running sum, rescaling of the output accumulator) then
// lives in that lane; only one exchange with lane ^ 32 (the other 16 keys of
// the same query) is needed per tile.  The output is accumulated transposed
// as well, O^T = V^T . P^T, so P goes from accumulator registers straight
// into the MFMA "B" operand without leaving the lane; V is read from a
// [dh, L] (key-contiguous) layout so that its fragments are plain vector
// loads too.  K and V^T tiles are staged in LDS once per workgroup and shared
// by all waves, i.e. by all heads of the K/V group.
#include <algorithm>
#include <atomic>

#include "attention.hpp"
#include "attention_dev.hpp"
#include "xcd_deal.hpp"

namespace sf {

constexpr int NWAVE = 4;
constexpr int BKEY = 64;          // keys per LDS tile (two 32-key MFMA blocks)
#define SF_SCORE_OCC __attribute__((amdgpu_waves_per_eu(4, 4)))

// List of the 64-key tiles of [jbeg, jend) that contain at least one allowed key (ascending),
// built by the first wave; returns the count through *n_tiles.  Needs `words` complete.
__device__ __forceinline__ void build_tile_list(const uint32_t *words, int nwords, int jbeg, int jend,
                                                uint16_t *tiles, int *n_tiles)
{
    if (threadIdx.x < 64) {
        int base = 0;
        for (int t0 = jbeg / BKEY; t0 * BKEY < jend; t0 += 64) {
            const int t = t0 + (int)threadIdx.x;
            bool live = false;
            if (t * BKEY < jend) {
                const uint32_t w0 = words[2 * t], w1 = (2 * t + 1 < nwords) ? words[2 * t + 1] : 0u;
                live = (w0 | w1) != 0u;
            }
            const unsigned long long bal = __ballot(live);
            if (live) tiles[base + __popcll(bal & ((1ull << threadIdx.x) - 1ull))] = (uint16_t)t;
            base += __popcll(bal);
        }
        if (threadIdx.x == 0) *n_tiles = base;
    }
}

// K tile chunks of this thread -> registers (rows at or beyond L are zero); NT
// threads share a tile.  j0 must be wave-uniform: the tile base stays scalar
// and each lane adds a 32-bit offset that does not change from tile to tile.
template <int DH, int NT>
struct KTile {
    static constexpr int CH = DH / 8, TOTAL = BKEY * CH, N = (TOTAL + NT - 1) / NT;
    static __device__ __forceinline__ void fetch(const h16 *Kb, int64_t sl, int j0, int L, uint4 (&r)[N])
    {
        const char *base = reinterpret_cast<const char *>(Kb + (int64_t)j0 * sl);
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int c = threadIdx.x + u * NT;
            const int row = c / CH, cc = c % CH;
            const uint32_t off = (uint32_t)row * (uint32_t)sl * 2u + (uint32_t)cc * 16u;   // < 64 rows * row stride bytes
            const bool whole = j0 + BKEY <= L;                                             // uniform: all but a ragged last tile
            r[u] = make_uint4(0, 0, 0, 0);
            if ((TOTAL % NT == 0 || c < TOTAL) && (whole || j0 + row < L)) r[u] = *reinterpret_cast<const uint4 *>(base + off);
        }
    }
    static __device__ __forceinline__ void put(const uint4 (&r)[N], h16 *Ks)
    {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int c = threadIdx.x + u * NT;
            if (TOTAL % NT == 0 || c < TOTAL)
                *reinterpret_cast<uint4 *>(Ks + (c / CH) * (DH + PAD) + (c % CH) * 8) = r[u];
        }
    }
};

// ------------------------------------------------------------- sparsity score
// M_i = max_j s_ij - mean_j s_ij over allowed keys.  The max comes from the
// streamed S^T tiles; the mean is q_i . mean_key (computed once per group),
// which is the same number up to fp32 rounding.
// 1-D grid over (query block, sample*head) items, query block fastest; each
// wave owns QBS blocks of 32 queries.  The launch index is folded so that all
// query blocks of one (sample, head) - and of the neighbouring heads, which
// mostly share the K/V group - run on one XCD and find K in its L2.  K tiles
// are double-buffered in LDS and the next tile is prefetched into registers
// while the current one is multiplied, so one barrier per tile suffices.
// `parts` > 1: an item is also one range of key tiles (launches with few items: one 512-token sample and six heads are 12
// items that walk eight tiles one after the other, 9.5 us; as 96 items of one tile 5.2 us).  Then plane p of `score`
// receives the largest product of range p (-inf: no allowed key there) and plane `parts` the product with the mean key:
// subtracting before the ranges are joined would turn infinities of one range into the answer of another.
template <int DH, int QBS>
__global__ __launch_bounds__(NWAVE * 64) SF_SCORE_OCC void score_bf16_kernel(
    const h16 *__restrict__ Q, sf_strides sq, const h16 *__restrict__ K, sf_strides sk,
    const int32_t *__restrict__ head_group, int hg_stride, const int32_t *__restrict__ pattern_id,
    const uint8_t *__restrict__ query_valid, const uint8_t *__restrict__ key_mask,
    const float *__restrict__ stats, int nH, int nG, int L, int Lk, float *__restrict__ score, int scoreH,
    int qblocks, int n_items, int parts, int64_t part_stride, const int32_t *__restrict__ row0,
    const int32_t *__restrict__ row0_k)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    h16 *Ks = reinterpret_cast<h16 *>(smem);                              // [2][BKEY][DH+PAD]
    float *kbar = reinterpret_cast<float *>(Ks + 2 * BKEY * (DH + PAD));        // [DH]
    uint32_t *words = reinterpret_cast<uint32_t *>(kbar + DH);                  // [ceil(Lk/32)]
    uint16_t *tiles = reinterpret_cast<uint16_t *>(words + (Lk + 31) / 32);     // [ceil(Lk/64)]
    __shared__ int n_tiles;

    const int item = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (item >= n_items) return;                          // uniform
    const int qblk = item % qblocks, part = (item / qblocks) % parts, bh = item / (qblocks * parts), b = bh / nH, h = bh % nH;
    const int g = head_group[(int64_t)(pattern_id ? pattern_id[b] : 0) * hg_stride + h];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lhi = lane >> 5;
    const uint8_t *kv = query_valid ? query_valid + (int64_t)b * L : nullptr;
    const int nwords = (Lk + 31) / 32;
    build_mask_words(key_mask ? key_mask + (int64_t)b * Lk : nullptr, Lk, words, nwords);
    if (threadIdx.x < DH) kbar[threadIdx.x] = stats[((int64_t)b * nG + g) * 2 * DH + threadIdx.x];

    // packed samples: Q (and K, unless it is the gathered key sample of the workspace) start at the sample's own row
    const h16 *Qb = Q + sample_offset(row0, b, sq) + (int64_t)h * sq.h;
    const h16 *Kb = K + sample_offset(row0_k, b, sk) + (int64_t)g * sk.h;
    const int q0 = (qblk * NWAVE + wave) * QBS * 32;

    h16x8 qf[QBS][DH / 16];
    float rmax[QBS];
#pragma unroll
    for (int qq = 0; qq < QBS; ++qq) {
        const int i = min(q0 + qq * 32 + l32, L - 1);
#pragma unroll
        for (int kk = 0; kk < DH / 16; ++kk)
            qf[qq][kk] = *reinterpret_cast<const h16x8 *>(Qb + (int64_t)i * sq.l + kk * 16 + lhi * 8);
        rmax[qq] = -INFINITY;
    }
    __syncthreads();
    const int kpp = ((Lk + BKEY - 1) / BKEY + parts - 1) / parts * BKEY;            // keys per part
    build_tile_list(words, nwords, part * kpp, min(Lk, (part + 1) * kpp), tiles, &n_tiles);
    __syncthreads();
    const int nt = n_tiles;

    using KT_ = KTile<DH, NWAVE * 64>;
    uint4 kreg[KT_::N];
    auto tile_j0 = [&](int it) { return __builtin_amdgcn_readfirstlane((int)tiles[it]) * BKEY; };   // same for every lane
    if (nt > 0) KT_::fetch(Kb, sk.l, tile_j0(0), Lk, kreg);
    for (int it = 0; it < nt; ++it) {
        const int j0 = tile_j0(it);
        h16 *Kt = Ks + (it & 1) * BKEY * (DH + PAD);
        KT_::put(kreg, Kt);
        __syncthreads();        // tile `it` visible; everyone is done with tile it-1 (the other buffer)
        if (it + 1 < nt) KT_::fetch(Kb, sk.l, tile_j0(it + 1), Lk, kreg);
        // the mask words are the same for every lane: keep them scalar
        const uint32_t w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)words[j0 / 32]);
        const uint32_t w1 = (j0 / 32 + 1 < nwords) ? (uint32_t)__builtin_amdgcn_readfirstlane((int)words[j0 / 32 + 1]) : 0u;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const uint32_t w = kb ? w1 : w0;
            if (w == 0u) continue;
            h16x8 kf[DH / 16];
#pragma unroll
            for (int kk = 0; kk < DH / 16; ++kk)
                kf[kk] = *reinterpret_cast<const h16x8 *>(Kt + (kb * 32 + l32) * (DH + PAD) + kk * 16 + lhi * 8);
            if (w == 0xffffffffu) {                 // scalar branch: the usual tile, no masking
#pragma unroll
                for (int qq = 0; qq < QBS; ++qq) {
                    f32x16 s;
#pragma unroll
                    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
                    for (int kk = 0; kk < DH / 16; ++kk)
                        s = SF_MFMA16(kf[kk], qf[qq][kk], s, 0, 0, 0);
                    float m = rmax[qq];
#pragma unroll
                    for (int e = 0; e < 16; e += 2) m = fmaxf(fmaxf(m, s[e]), s[e + 1]);
                    rmax[qq] = m;
                }
            } else {
                const uint32_t wl = w >> (lhi * 4);
#pragma unroll
                for (int qq = 0; qq < QBS; ++qq) {
                    f32x16 s;
#pragma unroll
                    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
                    for (int kk = 0; kk < DH / 16; ++kk)
                        s = SF_MFMA16(kf[kk], qf[qq][kk], s, 0, 0, 0);
                    float m = rmax[qq];
#pragma unroll
                    for (int e = 0; e < 16; ++e)       // key row of s[e]: (e/4)*8 + lhi*4 + e%4
                        m = fmaxf(m, ((wl >> ((e / 4) * 8 + (e % 4))) & 1u) ? s[e] : -INFINITY);
                    rmax[qq] = m;
                }
            }
        }
    }

    const float scale = 1.0f / sqrtf((float)DH);
#pragma unroll
    for (int qq = 0; qq < QBS; ++qq) {
        float m = fmaxf(rmax[qq], __shfl_xor(rmax[qq], 32));
        float dot = 0.f;
#pragma unroll
        for (int kk = 0; kk < DH / 16; ++kk)
#pragma unroll
            for (int e = 0; e < 8; ++e) dot = fmaf((float)qf[qq][kk][e], kbar[kk * 16 + lhi * 8 + e], dot);
        dot += __shfl_xor(dot, 32);
        const int i = q0 + qq * 32 + l32;
        if (lhi == 0 && i < L) {
            const bool ok = !kv || kv[i];
            float *out = score + ((int64_t)b * scoreH + h) * L + i;
            if (parts > 1) {                              // the selection sees every range: it takes mean, scale and mask
                out[part * part_stride] = m;
                if (part == 0) out[parts * part_stride] = dot;
            } else {
                *out = !ok ? -INFINITY : nt == 0 ? 0.f : (m - dot) * scale;      // no allowed key scores 0
            }
        }
    }
}

// ---------------------------------------------------------------- active pass
// A "pair" is (head of the group, block of 32 active queries).  A workgroup of
// AWAVE waves serves one (sample, K/V group, key split): each wave owns a
// pair and all waves share the K / V^T tiles staged in LDS; a group with more
// pairs than AWAVE is served in several passes over the key range.
// 1-D grid; the launch index is folded so that consecutive work items (the
// pair chunks of one (sample, group), which read the same K/V) run on the same
// XCD and share its L2, and the items are spread evenly over the XCDs.
constexpr int AWAVE = 8;

// NW = waves per workgroup.  Four instead of eight where a (sample, group) has at most four pairs: the same registers
// per wave then leave room for three workgroups per compute unit, and no wave is without a pair.
// Many active rows (dense-like patterns): at 126 registers (dh 64; 102 at dh 32) two workgroups share a compute unit, and one runs
// its softmax on the vector ALU while the other has the matrix pipe.  (128 are the limit for that.  As a minimum in the launch
// bounds it makes the compiler spill, so a test of the build watches the number.)  us for this launch, every query active, a
// kernel of two query blocks per wave that kept the waves of a SIMD in opposite phases by barriers, one workgroup per compute
// unit / this: 16 samples of 4096 keys, 8 heads 696 / 710; 8 of 1777 82 / 82; 1 of 4096, 4 heads 143 / 101; 64 of 1500, 3 heads of
// dh 32 165 / 124; 32 of 512, 4 heads 29 / 22; 4 of 1024, 4 heads 44 / 30.  Few long problems gain, many are level: there the
// calls gained by statistics that are not formed and a faster transposition (746 / 731, 109 / 95).
template <int DH, int NW>
__global__ __launch_bounds__(NW * 64) void attend_bf16_kernel(
    const h16 *__restrict__ Q, sf_strides sq, const h16 *__restrict__ K, sf_strides sk,
    const h16 *__restrict__ VT, sf_strides svt, const int32_t *__restrict__ head_group, int hg_stride,
    const int32_t *__restrict__ pattern_id, const uint8_t *__restrict__ key_valid,
    const int32_t *__restrict__ sel, int selH, int nH, int nG, int BG, int chunks, int L, int Lp, int U,
    int Upad, int splits, int keys_per_split, h16 *__restrict__ O, int64_t ldo,
    float *__restrict__ part_o, float *__restrict__ part_ml, const int32_t *__restrict__ row0)
{
    constexpr int NT = NW * 64;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int KT = BKEY * (DH + PAD), VT_ = DH * (BKEY + PAD);          // elements of one K / V^T tile
    h16 *Ks = reinterpret_cast<h16 *>(smem);                         // [2][BKEY][DH+PAD]
    h16 *Vs = Ks + 2 * KT;                                              // [2][DH][BKEY+PAD]
    uint32_t *words = reinterpret_cast<uint32_t *>(Vs + 2 * VT_);          // [ceil(L/32)]
    uint16_t *tiles = reinterpret_cast<uint16_t *>(words + (L + 31) / 32); // [ceil(L/64)]
    __shared__ int heads[64];
    __shared__ int n_heads, n_tiles;

    // launch index -> work item: XCD x (launch index % 8) takes the x-th eighth of the items
    const int per_xcd = gridDim.x / 8;
    const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (item >= chunks * BG * splits) return;             // uniform
    const int chunk = item % chunks, sp = item / (chunks * BG);
    int bg = (item / chunks) % BG;
    // Masked samples differ in cost: each XCD gets one of every eight problems instead of neighbours, which are one sample's groups.
    // us a call, neighbours / so, kernel otherwise the same but for the first pair: 8 samples of 1777 keys in 4 groups, half of
    // them at random with a modality missing, pass 79.0 / 76.8; 16 of 1500 in 4 groups, every second one so, 126 / 117 (132 with
    // the same one of every eight, which is always an odd or always an even sample).
    if (key_valid && BG % 8 == 0) bg = deal(bg / (BG / 8), bg % (BG / 8));
    const int b = bg / nG, g = bg % nG;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lhi = lane >> 5;
    const int32_t *hg = head_group + (int64_t)(pattern_id ? pattern_id[b] : 0) * hg_stride;

    if (wave == 0) {                      // ordered list of the group's heads (nH <= 64)
        const bool mine = lane < nH && hg[lane] == g;
        const unsigned long long bal = __ballot(mine);
        if (mine) heads[__popcll(bal & ((1ull << lane) - 1ull))] = lane;
        if (lane == 0) n_heads = __popcll(bal);
    }
    const uint8_t *kv = key_valid ? key_valid + (int64_t)b * L : nullptr;
    const int nwords = (L + 31) / 32;
    build_mask_words(kv, L, words, nwords);
    const int jbeg = sp * keys_per_split, jend = min(L, jbeg + keys_per_split);
    __syncthreads();
    build_tile_list(words, nwords, jbeg, jend, tiles, &n_tiles);
    __syncthreads();
    const int nt = n_tiles;
    const int nqb = Upad / 32;
    const int npairs = n_heads * nqb;

    const h16 *Kb = K + sample_offset(row0, b, sk) + (int64_t)g * sk.h;
    const h16 *Vb = VT + (int64_t)b * svt.b + (int64_t)g * svt.h;        // the transposed V is always b-strided
    const float sc = LOG2E / sqrtf((float)DH);

    // V^T tile chunks of this thread -> registers; keys at or beyond L are zeroed
    constexpr int VTOTAL = DH * (BKEY / 8), NV = (VTOTAL + NT - 1) / NT;
    auto fetch_v = [&](int j0, uint4 (&r)[NV]) {
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int c = threadIdx.x + u * NT;
            const int e = c / (BKEY / 8), cc = c % (BKEY / 8);
            const int j = j0 + cc * 8;
            uint4 v = make_uint4(0, 0, 0, 0);
            if ((VTOTAL % NT == 0 || c < VTOTAL) && (j0 + BKEY <= Lp || j < Lp)) {
                const uint32_t off = (uint32_t)e * (uint32_t)svt.l * 2u + (uint32_t)cc * 16u;   // < dh rows of Lp keys
                v = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(Vb + j0) + off);
            }
            r[u] = v;          // (keys at or beyond L are zeroed when the chunk is written to LDS: touching the value
                               // here would make the wave wait for the load it has just issued)
        }
    };
    auto put_v = [&](const uint4 (&r)[NV], h16 *Vt, int j0) {
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int c = threadIdx.x + u * NT;
            if (VTOTAL % NT == 0 || c < VTOTAL) {
                uint4 v = r[u];
                const int j = j0 + (c % (BKEY / 8)) * 8;
                if (j0 + BKEY > L && j + 8 > L) {      // last tile of a ragged row only
                    uint16_t *hv = reinterpret_cast<uint16_t *>(&v);
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (j + e >= L) hv[e] = 0;
                }
                *reinterpret_cast<uint4 *>(Vt + (c / (BKEY / 8)) * (BKEY + PAD) + (c % (BKEY / 8)) * 8) = v;
            }
        }
    };
    using KT_ = KTile<DH, NT>;
    auto tile_j0 = [&](int it) { return __builtin_amdgcn_readfirstlane((int)tiles[it]) * BKEY; };   // same for every lane

    for (int pair0 = chunk * NW; pair0 < npairs; pair0 += chunks * NW) {
        // When this pass has pairs for at most half of the waves (few active rows: U = c*ceil(ln L) gives one or two
        // blocks of 32 per head), the others would only help with the staging: instead KG groups of waves take the
        // same pairs and every KG-th key tile each, and their partial results are merged through LDS at the end.
        int kg = 1;
        {
            const int waves_used = min(npairs - pair0, NW);
            // only where the launch is short of workgroups (the host split the keys for that reason): with a
            // (sample, group) problem per compute unit or more the idle waves cost nothing and the merge does
            while (splits > 1 && waves_used * kg * 2 <= NW) kg *= 2;
        }
        const int pslots = NW / kg;                  // waves that hold distinct pairs
        const int pw = wave % pslots, kgi = wave / pslots;
        int head, qidx, slot;
        auto locate = [&](int lane32) {
            const int pi = pair0 + pw;
            head = -1; qidx = -1; slot = 0;
            if (pi < npairs) {
                head = heads[pi / nqb];
                slot = (pi % nqb) * 32 + lane32;
                if (slot < U) qidx = sel[((int64_t)b * selH + head) * U + slot];
            }
        };
        locate(l32);
        const h16 *qrow = Q + sample_offset(row0, b, sq) + (int64_t)max(head, 0) * sq.h + (int64_t)max(qidx, 0) * sq.l;
        h16x8 qf[DH / 16];
#pragma unroll
        for (int kk = 0; kk < DH / 16; ++kk) qf[kk] = *reinterpret_cast<const h16x8 *>(qrow + kk * 16 + lhi * 8);
        // no pair, or none of its slots names a row (masked queries leave whole blocks empty): uniform over the wave
        const bool idle = __builtin_amdgcn_ballot_w64(qidx >= 0) == 0ull;
        if (!__syncthreads_or(!idle)) continue;               // nobody in the workgroup has one

        f32x16 oacc[DH / 32];
        float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
        for (int db = 0; db < DH / 32; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[db][e] = 0.f;

        uint4 kreg[KT_::N], vreg[NV];
        if (nt > 0) { KT_::fetch(Kb, sk.l, tile_j0(0), L, kreg); fetch_v(tile_j0(0), vreg); }

        for (int it = 0; it < nt; ++it) {
            const int j0 = tile_j0(it);
            h16 *Kt = Ks + (it & 1) * KT, *Vt = Vs + (it & 1) * VT_;
            KT_::put(kreg, Kt);
            put_v(vreg, Vt, j0);
            __syncthreads();        // tile `it` visible; everyone is done with tile it-1 (the other buffers)
            if (it + 1 < nt) { const int jn = tile_j0(it + 1); KT_::fetch(Kb, sk.l, jn, L, kreg); fetch_v(jn, vreg); }
            if (idle || (it & (kg - 1)) != kgi) continue;          // not this wave's tile
            const uint32_t w0 = words[j0 / 32], w1 = (j0 / 32 + 1 < nwords) ? words[j0 / 32 + 1] : 0u;
            // the same for every lane: a tile with all 64 keys allowed skips the masking
            const bool all_allowed = (uint32_t)__builtin_amdgcn_readfirstlane((int)(w0 & w1)) == 0xffffffffu;

            // S^T blocks for the two 32-key halves
            f32x16 s[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                h16x8 kf[DH / 16];
#pragma unroll
                for (int kk = 0; kk < DH / 16; ++kk)
                    kf[kk] = *reinterpret_cast<const h16x8 *>(Kt + (kb * 32 + l32) * (DH + PAD) + kk * 16 + lhi * 8);
#pragma unroll
                for (int e = 0; e < 16; ++e) s[kb][e] = 0.f;
#pragma unroll
                for (int kk = 0; kk < DH / 16; ++kk) s[kb] = SF_MFMA16(kf[kk], qf[kk], s[kb], 0, 0, 0);
            }

            // online softmax per query (per lane), log2 domain
            if (!all_allowed) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    const uint32_t wl = (kb ? w1 : w0) >> (lhi * 4);
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (!((wl >> ((e / 4) * 8 + (e % 4))) & 1u)) s[kb][e] = -INFINITY;
                }
            }
            float mt = fmaxf(fmaxf(s[0][0], s[0][1]), s[1][0]);
            mt = fmaxf(fmaxf(mt, s[1][1]), s[0][2]);
#pragma unroll
            for (int e = 3; e < 15; e += 2) mt = fmaxf(fmaxf(mt, s[0][e]), s[0][e + 1]);
#pragma unroll
            for (int e = 2; e < 16; e += 2) mt = fmaxf(fmaxf(mt, s[1][e]), s[1][e + 1]);
            mt = fmaxf(mt, s[0][15]) * sc;             // sc > 0: max and scaling commute
            mt = both_halves_max(mt);                  // the other 16 keys of each 32-key block sit in lane ^ 32
            // The reference m_run of the exponentials only has to stay within 2^RESCALE_LOG2 of the true running
            // maximum (sums and outputs are relative to the same reference, so the result does not depend on
            // it): it moves, and the accumulators are rescaled, only when some query of the wave needs it.
            // After the first tiles of a row that is rare, which removes the rescaling from the common path.
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(mt > m_run + RESCALE_LOG2) != 0ull, 0)) {
                const float m_new = fmaxf(m_run, mt);
                const float alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.f : m_new));
                m_run = m_new;
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < DH / 32; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
            }
            const float nm = m_run == -INFINITY ? 0.f : -m_run;
            float rs0 = 0.f, rs1 = 0.f;
            h16x8 pf[4];
            // k-step t covers keys 16t..16t+15; this lane supplies keys
            // {16t + lhi*4 + 0..3, 16t + 8 + lhi*4 + 0..3} = accumulator entries (t%2)*8 + 0..7 of block t/2
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int e = 0; e < 16; e += 2) {
                    const float p0 = __builtin_amdgcn_exp2f(fmaf(s[kb][e], sc, nm));
                    const float p1 = __builtin_amdgcn_exp2f(fmaf(s[kb][e + 1], sc, nm));
                    rs0 += p0;
                    rs1 += p1;
                    reinterpret_cast<uint32_t *>(&pf[kb * 2 + e / 8])[(e % 8) / 2] = pack2_h16(p0, p1);
                }
            l_run += rs0 + rs1;

            // O^T += V^T . P^T
#pragma unroll
            for (int db = 0; db < DH / 32; ++db) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const h16 *vrow = Vt + (db * 32 + l32) * (BKEY + PAD) + t * 16 + lhi * 4;
                    const h16x4 lo = *reinterpret_cast<const h16x4 *>(vrow);
                    const h16x4 hi = *reinterpret_cast<const h16x4 *>(vrow + 8);
                    h16x8 vf;
#pragma unroll
                    for (int e = 0; e < 4; ++e) { vf[e] = lo[e]; vf[4 + e] = hi[e]; }
                    oacc[db] = SF_MFMA16(vf, pf[t], oacc[db], 0, 0, 0);
                }
            }
        }

        // merge of the key groups: in log2(KG) rounds the upper half of the groups hands its running reference, sum
        // and accumulator over through the tile buffers (free now) and the lower half folds them into its own
        if (kg > 1) {
            float *mrg = reinterpret_cast<float *>(smem);              // [writer wave][DH/2 + 2][64 lanes]
            constexpr int PER = (DH / 32) * 16 + 2;
            static_assert((NW / 2) * PER * 64 * 4 <= 2 * KT * 2 + 2 * VT_ * 2, "merge scratch must fit in the tile buffers");
            for (int step = kg / 2; step >= 1; step /= 2) {
                __syncthreads();                                       // tile buffers (or the last round's slots) are free
                if (kgi >= step && kgi < 2 * step) {
                    float *dst = mrg + (size_t)(wave - step * pslots) * PER * 64 + lane;
#pragma unroll
                    for (int db = 0; db < DH / 32; ++db)
#pragma unroll
                        for (int e = 0; e < 16; ++e) dst[(db * 16 + e) * 64] = oacc[db][e];
                    dst[(DH / 32) * 16 * 64] = m_run;
                    dst[((DH / 32) * 16 + 1) * 64] = l_run;
                }
                __syncthreads();
                if (kgi < step) {
                    const float *src = mrg + (size_t)wave * PER * 64 + lane;
                    const float m_o = src[(DH / 32) * 16 * 64], l_o = src[((DH / 32) * 16 + 1) * 64];
                    const float m_new = fmaxf(m_run, m_o);
                    const float m_safe = m_new == -INFINITY ? 0.f : m_new;
                    const float a_me = __builtin_amdgcn_exp2f(m_run - m_safe), a_o = __builtin_amdgcn_exp2f(m_o - m_safe);
                    m_run = m_new;
                    l_run = l_run * a_me + l_o * a_o;
#pragma unroll
                    for (int db = 0; db < DH / 32; ++db)
#pragma unroll
                        for (int e = 0; e < 16; ++e) oacc[db][e] = oacc[db][e] * a_me + src[(db * 16 + e) * 64] * a_o;
                }
            }
        }

        // lane owns query l32 and output dims db*32 + ig*8 + lhi*4 + {0..3}
        const float l_tot = both_halves_sum(l_run);
        int lane32 = l32;
        asm volatile("" : "+v"(lane32));     // the row is looked up again: live across the loop it costs registers
        locate(lane32);
        if (qidx >= 0 && kgi == 0) {
            if (splits <= 1) {
                const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
                h16 *orow = O + (sample_row(row0, b, L) + qidx) * ldo + (int64_t)head * DH;
#pragma unroll
                for (int db = 0; db < DH / 32; ++db)
#pragma unroll
                    for (int ig = 0; ig < 4; ++ig) {
                        h16x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = (h16)(oacc[db][ig * 4 + e] * inv);
                        *reinterpret_cast<h16x4 *>(orow + db * 32 + ig * 8 + lhi * 4) = o;
                    }
            } else {
                const int64_t base = (((int64_t)b * nH + head) * splits + sp) * Upad + slot;   // [b, head, split, slot]
                float *po = part_o + base * DH;
#pragma unroll
                for (int db = 0; db < DH / 32; ++db)
#pragma unroll
                    for (int ig = 0; ig < 4; ++ig) {
                        f32x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = oacc[db][ig * 4 + e];
                        *reinterpret_cast<f32x4 *>(po + db * 32 + ig * 8 + lhi * 4) = o;
                    }
                if (lhi == 0) {
                    part_ml[base * 2] = m_run;
                    part_ml[base * 2 + 1] = l_tot;
                }
            }
        }
        __syncthreads();            // the next pass restages both tile buffers
    }
}

// ------------------------------------------------- active pass, few active rows (U < 256)
// A workgroup serves one (sample, head, block of 32 active queries) with the keys dealt to its waves in tiles of 32: wave w
// takes every NW-th live tile, reads its K and V^T fragments straight from memory into registers - no LDS, no barrier, no
// wait on another wave - and keeps a running softmax of its own; the NW partial results are merged through LDS at the
// end.  U = c * ceil(ln L) gives one or two blocks of 32 queries per head, so K and V of a group are read only a few
// times (from L2), and what counts is that every wave of every compute unit has loads in flight: staging the tiles in LDS
// for all heads of a group walked them one after the other in one workgroup per (sample, group).  us, staged (with the
// merge launch where the keys were split) / sliced: 256 samples of 480 keys, 4 heads 38 / 29; 64 of 384 keys, 6 heads
// 11.6 / 8.0; 37 of 1021 keys, 8 heads 20 + 7 / 18; 16 of 4096 keys, 8 heads 31 + 6 / 37; 1 of 512 keys, 6 heads 10 + 4 / 8.5;
// but 128 of 512 keys, 6 heads in two groups 19 / 23, 4 of 16384 keys, 2 heads in a group 16 + 5 / 118: attend_bf16_staged()
// chooses.
//
// The keys of a tile are assigned to the rows of S^T so that a lane's 16 scores are two runs of 8 consecutive keys: row
// 8 a + 4 h + r (a < 4, h < 2, r < 4) holds key 16 (a / 2) + 8 h + 4 (a % 2) + r.  P then meets V^T fragments that are
// 16 contiguous bytes.
template <int DH, int QB, int NW>
__global__ __launch_bounds__(NW * 64, DH == 128 || QB * DH == 128 ? 2 : 3) void attend_slice_bf16_kernel(
    const h16 *__restrict__ Q, sf_strides sq, const h16 *__restrict__ K, sf_strides sk,
    const h16 *__restrict__ VT, sf_strides svt, const int32_t *__restrict__ head_group, int hg_stride,
    const int32_t *__restrict__ pattern_id, const uint8_t *__restrict__ key_valid,
    const int32_t *__restrict__ sel, int selH, int nH, int nG, int nqb, int n_items, int L, int Lp, int U,
    h16 *__restrict__ O, int64_t ldo, const int32_t *__restrict__ row0)
{
    constexpr int KF = DH / 16, DB = DH / 32, OP = DH + 4;                // fragments of K, dim blocks, row of a partial
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float *part = reinterpret_cast<float *>(smem);                        // [NW][32][OP], one query block at a time
    float2 *ml = reinterpret_cast<float2 *>(part + NW * 32 * OP);         // [NW][QB * 32] reference, sum
    int32_t *rows = reinterpret_cast<int32_t *>(ml + NW * QB * 32);       // [QB * 32] query of a slot
    uint32_t *words = reinterpret_cast<uint32_t *>(rows + QB * 32);       // [ceil(L/32)] when there is a mask

    const int item = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (item >= n_items) return;                                          // uniform
    const int qb = item % nqb, bh = item / nqb, b = bh / nH, h = bh % nH;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, lhi = lane >> 5;
    int qidx[QB];
#pragma unroll
    for (int qq = 0; qq < QB; ++qq) {
        const int slot = (qb * QB + qq) * 32 + l32;
        qidx[qq] = slot < U ? sel[((int64_t)b * selH + h) * U + slot] : -1;
    }
    const int g = head_group[(int64_t)(pattern_id ? pattern_id[b] : 0) * hg_stride + h];
    const int nt = (L + 31) / 32;
    if (key_valid) build_mask_words(key_valid + (int64_t)b * L, L, words, nt);
    h16x8 qf[QB][KF];
#pragma unroll
    for (int qq = 0; qq < QB; ++qq) {
        if (threadIdx.x < 32) rows[qq * 32 + threadIdx.x] = qidx[qq];
        const h16 *qrow = Q + sample_offset(row0, b, sq) + (int64_t)h * sq.h + (int64_t)max(qidx[qq], 0) * sq.l;
#pragma unroll
        for (int kk = 0; kk < KF; ++kk) qf[qq][kk] = *reinterpret_cast<const h16x8 *>(qrow + kk * 16 + lhi * 8);
    }
    if (key_valid) __syncthreads();
    bool any = qidx[0] >= 0;              // a caller's list may hold its rows behind a block without any
#pragma unroll
    for (int qq = 1; qq < QB; ++qq) any |= qidx[qq] >= 0;
    if (__builtin_amdgcn_ballot_w64(any) == 0ull) return;                 // uniform over the workgroup: no row in these blocks

    const h16 *Kb = K + sample_offset(row0, b, sk) + (int64_t)g * sk.h + lhi * 8;
    const h16 *Vb = VT + (int64_t)b * svt.b + (int64_t)g * svt.h + (int64_t)l32 * svt.l + lhi * 8;
    const int krow = 16 * (l32 >> 4) + 8 * ((l32 >> 2) & 1) + 4 * ((l32 >> 3) & 1) + (l32 & 3);
    const float sc = LOG2E / sqrtf((float)DH);
    auto word = [&](int t) -> uint32_t {                                  // allowed keys of tile t
        if (key_valid) return (uint32_t)__builtin_amdgcn_readfirstlane((int)words[t]);
        return t * 32 + 32 <= L ? 0xffffffffu : (1u << (L - t * 32)) - 1u;
    };
    // the wave's next tile: the live ones are dealt round-robin
    int blk = -64, turn = 0;
    unsigned long long live = 0ull;
    auto next = [&]() -> int {
        for (;;) {
            while (!live) {
                blk += 64;
                if (blk >= nt) return -1;
                live = __builtin_amdgcn_ballot_w64(blk + lane < nt && (!key_valid || words[blk + lane] != 0u));
            }
            const int t = blk + __ffsll((long long)live) - 1;
            live &= live - 1ull;
            const bool mine = turn == wave;
            turn = turn + 1 == NW ? 0 : turn + 1;
            if (mine) return t;
        }
    };
    struct KV { h16x8 k[KF], v[DB][2]; };
    auto load = [&](KV &x, int t) {
        const h16 *kp = Kb + (int64_t)min(t * 32 + krow, L - 1) * sk.l;   // rows beyond L: masked
#pragma unroll
        for (int kk = 0; kk < KF; ++kk) x.k[kk] = *reinterpret_cast<const h16x8 *>(kp + kk * 16);
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int p = 0; p < 2; ++p)
                x.v[d][p] = *reinterpret_cast<const h16x8 *>(Vb + (int64_t)(d * 32) * svt.l + min(t * 32 + p * 16, Lp - 8 - lhi * 8));
    };
    f32x16 o[QB][DB];
    float m_run[QB], l_run[QB];
#pragma unroll
    for (int qq = 0; qq < QB; ++qq) {
        m_run[qq] = -INFINITY;
        l_run[qq] = 0.f;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[qq][d][e] = 0.f;
    }
    auto process = [&](KV &x, int t) {
        f32x16 s[QB];
#pragma unroll
        for (int qq = 0; qq < QB; ++qq) {
#pragma unroll
            for (int e = 0; e < 16; ++e) s[qq][e] = 0.f;
#pragma unroll
            for (int kk = 0; kk < KF; ++kk) s[qq] = SF_MFMA16(x.k[kk], qf[qq][kk], s[qq], 0, 0, 0);
        }
        const uint32_t w = word(t);
        if (w != 0xffffffffu) {                                           // scalar branch
            const uint32_t wl = w >> (lhi * 8);                           // s[e]: key 16 (e / 8) + 8 lhi + e % 8
#pragma unroll
            for (int qq = 0; qq < QB; ++qq)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (!((wl >> ((e / 8) * 16 + e % 8)) & 1u)) s[qq][e] = -INFINITY;
            if (t * 32 + 32 > L) {                                        // V^T beyond L may hold anything
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (t * 32 + p * 16 + lhi * 8 + i >= L) x.v[d][p][i] = (h16)0.f;
            }
        }
        h16x8 pf[QB][2];
#pragma unroll
        for (int qq = 0; qq < QB; ++qq) {
            float mt = fmaxf(s[qq][0], s[qq][1]);
#pragma unroll
            for (int e = 2; e < 16; e += 2) mt = fmaxf(fmaxf(mt, s[qq][e]), s[qq][e + 1]);
            mt = both_halves_max(mt) * sc;                                // sc > 0: max and scaling commute
            // the reference of the exponentials moves only when some query exceeds it by 2^RESCALE_LOG2 (results are
            // relative to it and do not depend on it)
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(mt > m_run[qq] + RESCALE_LOG2) != 0ull, 0)) {
                const float m_new = fmaxf(m_run[qq], mt);
                const float alpha = __builtin_amdgcn_exp2f(m_run[qq] - (m_new == -INFINITY ? 0.f : m_new));
                m_run[qq] = m_new;
                l_run[qq] *= alpha;
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o[qq][d][e] *= alpha;
            }
            const float nm = m_run[qq] == -INFINITY ? 0.f : -m_run[qq];
            float rs0 = 0.f, rs1 = 0.f;
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const float p0 = __builtin_amdgcn_exp2f(fmaf(s[qq][e], sc, nm)), p1 = __builtin_amdgcn_exp2f(fmaf(s[qq][e + 1], sc, nm));
                rs0 += p0;
                rs1 += p1;
                reinterpret_cast<uint32_t *>(&pf[qq][e / 8])[(e % 8) / 2] = pack2_h16(p0, p1);
            }
            l_run[qq] += rs0 + rs1;
        }
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int qq = 0; qq < QB; ++qq) o[qq][d] = SF_MFMA16(x.v[d][p], pf[qq][p], o[qq][d], 0, 0, 0);
    };
    if constexpr (DH == 128) {                                            // no registers for a second tile
        KV x;
        for (int t = next(); t >= 0; t = next()) {
            load(x, t);
            process(x, t);
        }
    } else {
        KV x, y;
        int t = next();
        if (t >= 0) load(x, t);
        while (t >= 0) {                                                  // one tile ahead
            int u = next();
            if (u >= 0) load(y, u);
            process(x, t);
            if (u < 0) break;
            t = next();
            if (t >= 0) load(x, t);
            process(y, u);
        }
    }
    // merge: partial of wave w at part[w][query][dim]; lane owns query l32 and dims d*32 + q*8 + lhi*4 + {0..3}
#pragma unroll
    for (int qq = 0; qq < QB; ++qq) {
        const float l_tot = both_halves_sum(l_run[qq]);
        if (lhi == 0) ml[(wave * QB + qq) * 32 + l32] = make_float2(m_run[qq], l_tot);
        if (qq > 0) __syncthreads();                                      // the last block's partials have been read
        float *mine = part + (wave * 32 + l32) * OP + lhi * 4;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = o[qq][d][q * 4 + e];
                *reinterpret_cast<f32x4 *>(mine + d * 32 + q * 8) = v;
            }
        __syncthreads();
        constexpr int CPR = DH / 4;
        for (int c = threadIdx.x; c < 32 * CPR; c += NW * 64) {
            const int q = c / CPR, d4 = (c % CPR) * 4, qi = rows[qq * 32 + q];
            if (qi < 0) continue;
            float m = -INFINITY;
#pragma unroll
            for (int w = 0; w < NW; ++w) m = fmaxf(m, ml[(w * QB + qq) * 32 + q].x);
            const float m_safe = m == -INFINITY ? 0.f : m;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            float den = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float2 t = ml[(w * QB + qq) * 32 + q];
                const float wgt = __builtin_amdgcn_exp2f(t.x - m_safe);
                den += wgt * t.y;
                const f32x4 v = *reinterpret_cast<const f32x4 *>(part + (w * 32 + q) * OP + d4);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += wgt * v[e];
            }
            const float inv = den > 0.f ? 1.0f / den : 0.f;
            h16x4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = (h16)(acc[e] * inv);
            *reinterpret_cast<h16x4 *>(O + (sample_row(row0, b, L) + qi) * ldo + (int64_t)h * DH + d4) = out;
        }
    }
}

// ---------------------------------------------------------------- host side
template <int DH, int QBS>
static int32_t launch_score(const AttnArgs &a, const void *Kx, sf_strides skx, int Lk, const uint8_t *key_mask,
                            const float *stats, float *score, int scoreH, int parts, hipStream_t st)
{
    const size_t lds = (size_t)2 * BKEY * (DH + PAD) * 2 + DH * 4 + (size_t)ceil_div(Lk, 32) * 4 +
                       (size_t)ceil_div(Lk, BKEY) * 2 + 16;
    const int qblocks = ceil_div(a.L, NWAVE * QBS * 32);
    const int64_t items = (int64_t)qblocks * a.B * a.nH * parts;
    if (items > (1 << 30)) return fail(SF_ERR_SHAPE, "sparse_gqa(bf16): too many work items");
    dim3 grid((unsigned)align_up(items, 8));
    ProfScope prof(SF_KERNEL_SCORE, st);
    hipLaunchKernelGGL((score_bf16_kernel<DH, QBS>), grid, dim3(NWAVE * 64), lds, st, (const h16 *)a.Q,
                       a.sq, (const h16 *)Kx, skx, a.head_group, a.hg_stride, a.pattern_id, a.key_valid,
                       key_mask, stats, a.nH, a.nG, a.L, Lk, score, scoreH, qblocks, (int)items, parts,
                       (int64_t)a.B * scoreH * a.L, a.row0, Kx == a.K ? a.row0 : nullptr);
    return SF_OK;
}

static bool score_wide(const AttnArgs &a) { return a.L >= 1024; }

// With at least a workgroup per compute unit the stream is not split; below that, towards two per compute unit, down
// to one key tile each, and at most eight ways (the selection reads every part of a score).
int score_bf16_parts(const AttnArgs &a, int Lk)
{
    const int rows = NWAVE * 32 * (a.dh == 128 ? (score_wide(a) ? 2 : 1) : (score_wide(a) ? 4 : 2));      // per workgroup
    const int64_t items = (int64_t)ceil_div(a.L, rows) * a.B * a.nH;
    if (items >= 256) return 1;
    return (int)std::min<int64_t>(std::min(ceil_div(Lk, BKEY), 8), (512 + items - 1) / items);
}

int32_t score_bf16(const AttnArgs &a, const void *Kx, sf_strides skx, int Lk, const uint8_t *key_mask,
                   const float *stats, float *score, int scoreH, int parts, hipStream_t st)
{
    const bool wide = score_wide(a);
#define SF_SCORE_ARGS a, Kx, skx, Lk, key_mask, stats, score, scoreH, parts, st
    switch (a.dh) {
    case 32:  return wide ? launch_score<32, 4>(SF_SCORE_ARGS) : launch_score<32, 2>(SF_SCORE_ARGS);
    case 64:  return wide ? launch_score<64, 4>(SF_SCORE_ARGS) : launch_score<64, 2>(SF_SCORE_ARGS);
    case 128: return wide ? launch_score<128, 2>(SF_SCORE_ARGS) : launch_score<128, 1>(SF_SCORE_ARGS);
    }
#undef SF_SCORE_ARGS
    return fail(SF_ERR_SHAPE, "sparse_gqa(bf16): dh must be 32, 64 or 128");
}

// Waves of the staged kernel: four instead of eight where the launch has a (sample, group) problem per compute unit or
// more (no key splits) and at most four pairs per problem (256 samples of 480 keys, 4 heads of a group each: 66 -> 49 us);
// with split keys the launch is short of work per compute unit and eight waves with key groups are faster (45 -> 40 us for 16
// samples of 4096 keys, two heads per group); dh 128 needs 232 registers with four waves, i.e. one wave per SIMD, and so few
// pairs of dh 32 are served by the sliced kernel.
static int staged_waves(int dh, int pairs, int splits) { return dh == 64 && pairs <= 4 && splits == 1 ? 4 : AWAVE; }

// The sliced kernel: two query blocks per wave halve the reads of K and V (256 samples of 480 keys, 4 heads: 35 -> 29 us) where
// the heads alone fill the chip; four waves instead of eight where the items do.
struct SliceShape { int qb, nw; int64_t items; };
static SliceShape slice_shape(const AttnArgs &a)
{
    const int64_t heads = (int64_t)a.B * a.nH, nqb = ceil_div(a.U, 32);
    const int qb = a.dh < 128 && nqb > 1 && heads >= 256 ? 2 : 1;
    return SliceShape{qb, qb == 2 || heads * nqb >= 512 ? 4 : 8, heads * ((nqb + qb - 1) / qb)};
}

// Which kernel serves fewer than STAGED_U active rows.  Sliced, every item (head, query blocks) reads K and V for itself and
// one workgroup walks all its keys; staged, the pairs of a group share them and the keys of a sample are split over the
// compute units, at the price of a merge.  So sliced it is for short sequences, and where a group has one head or two;
// long ones (16384 keys, 4 heads: 118 us sliced, 17 + 5 staged) and groups of many pairs (512 samples of 512 keys,
// 16 heads in one group, dh 128: 538 / 206) stay with the staged tiles.
// Where nothing is split, few pairs are sliced, and with a (sample, group) problem per compute unit more of them are not;
// the rest is an estimate of both times in us (a chain of key tiles, longer where the workgroups need more than one round;
// or the traffic, each item's own where it is sliced).  Its constants are a fit to 2400 calls drawn at random (1 to 512
// samples of 48 to 16384 keys, 1 to 8 groups of 1 to 16 heads, 1 to 255 active rows, a third of them masked): over those the
// choice costs 0.4 % of a call against the better kernel, 20 % at worst (all sliced: 6 %, a factor of 1.9; all staged: 11 %,
// 2.1).  Since then the staged kernel has come to share a compute unit between two workgroups: over 110 calls of 1100 to 16384
// keys the choice costs 1.5 %, 13 % at worst (all sliced: 5.6 %, all staged: 5.5 %).
bool attend_bf16_staged(const AttnArgs &a, int splits)
{
    if (a.U >= STAGED_U) return true;
    struct Fit {
        double c, step8, step4, step2, room, room2;          // sliced: call, step of 32 keys (8 waves, 4, two query blocks), workgroups per compute unit
        double c_st, tile8, tile4, room8, room4, merge;      // staged: call, tile of 64 keys (8 waves, 4), workgroups per compute unit, merge launch
        double mb, mb_item;                                  // a megabyte of K and V from memory, and once more per item
    };
    static constexpr Fit f32 = {4.1, 0.76, 0.56, 0.29, 1.55, 1.25, 4.5, 0.27, 0.27, 0.41, 0.41, 6.1, 0.16, 0.024};
    static constexpr Fit f64 = {5.4, 1.40, 1.10, 0.85, 0.92, 0.67, 6.5, 0.96, 1.35, 0.53, 1.25, 3.8, 0.17, 0.071};
    static constexpr Fit f128 = {3.5, 2.98, 2.60, 2.60, 0.90, 0.90, 5.2, 1.45, 1.45, 0.59, 0.59, 5.9, 0.18, 0.080};
    const Fit &f = a.dh == 32 ? f32 : a.dh == 64 ? f64 : f128;
    const int64_t bg = (int64_t)a.B * a.nG;
    const int nqb = ceil_div(a.U, 32), per_group = ceil_div(a.nH, a.nG), pairs = per_group * nqb;
    if (splits == 1 && pairs <= (a.dh == 32 ? 6 : a.dh == 64 ? 2 : 1)) return false;
    if (bg >= 256) return true;
    const double mb = 4e-6 * bg * a.L * a.dh;
    const SliceShape s = slice_shape(a);
    const double step = s.qb == 2 ? f.step2 : s.nw == 4 ? f.step4 : f.step8, steps = ceil_div(ceil_div(a.L, 32), s.nw);
    const double sliced = f.c + std::max(step * steps * std::max(1.0, s.items * s.nw / (2048.0 * (s.qb == 2 ? f.room2 : f.room))),
                                         mb * (f.mb + f.mb_item * per_group * ((nqb + s.qb - 1) / s.qb)));
    const int nw = staged_waves(a.dh, pairs, splits);
    const double tiles = ceil_div(ceil_div(a.L, BKEY), splits), wgs = (double)ceil_div(pairs, nw) * bg * splits;
    const double staged = f.c_st + std::max(tiles * (nw == 4 ? f.tile4 : f.tile8) * std::max(1.0, wgs / (256.0 * (nw == 4 ? f.room4 : f.room8))), mb * f.mb) +
                          (splits > 1 ? f.merge : 0.0);
    return staged <= sliced;
}

template <int DH>
static int32_t launch_attend(const AttnArgs &a, const AttnPlan &pl, const void *vt, sf_strides svt,
                             const int32_t *sel, int selH, hipStream_t st)
{
    const size_t lds = (size_t)2 * BKEY * (DH + PAD) * 2 + (size_t)2 * DH * (BKEY + PAD) * 2 +
                       (size_t)ceil_div(a.L, 32) * 4 + (size_t)ceil_div(a.L, BKEY) * 2 + 16;
    const int nqb = pl.Upad / 32, BG = a.B * a.nG;
    // pair chunks per (sample, group) for evenly spread heads; a group with more heads takes several passes
    const int pairs = ceil_div(a.nH, a.nG) * nqb;
    const int nw = staged_waves(DH, pairs, pl.splits);
    const int chunks = ceil_div(pairs, nw);
    const int64_t items = (int64_t)chunks * BG * pl.splits;
    if (items > (1 << 30)) return fail(SF_ERR_SHAPE, "sparse_gqa(bf16): too many work items");
    dim3 grid((unsigned)align_up(items, 8));
    ProfScope prof(SF_KERNEL_ATTEND, st);
#define SF_ATTEND_ARGS grid, dim3(nw * 64), lds, st, (const h16 *)a.Q, a.sq, (const h16 *)a.K, a.sk, (const h16 *)vt, \
                       svt, a.head_group, a.hg_stride, a.pattern_id, a.key_valid, sel, selH, a.nH, a.nG, BG, chunks, a.L, \
                       pl.Lp, a.U, pl.Upad, pl.splits, pl.keys_per_split, (h16 *)a.O, a.ldo, pl.part_o, pl.part_ml, a.row0
    if (nw == 4) hipLaunchKernelGGL((attend_bf16_kernel<DH, DH == 64 ? 4 : AWAVE>), SF_ATTEND_ARGS);
    else hipLaunchKernelGGL((attend_bf16_kernel<DH, AWAVE>), SF_ATTEND_ARGS);
#undef SF_ATTEND_ARGS
    return SF_OK;
}

template <int DH, int QB, int NW>
static int32_t launch_attend_slice(const AttnArgs &a, const AttnPlan &pl, const void *vt, sf_strides svt, const int32_t *sel,
                                   int selH, hipStream_t st)
{
    auto kern = attend_slice_bf16_kernel<DH, QB, NW>;
    const size_t lds = (size_t)NW * 32 * (DH + 4) * 4 + (size_t)NW * QB * 32 * 8 + QB * 128 + (size_t)ceil_div(a.L, 32) * 4;
    static std::atomic<bool> attr_set{false};     // setting the attribute twice is harmless
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) !=
            hipSuccess)
            return fail(SF_ERR_HIP, "sparse_gqa: cannot reserve LDS for the active pass");
        attr_set = true;
    }
    const int nqb = ceil_div(pl.Upad / 32, QB);
    const int64_t items = (int64_t)a.B * a.nH * nqb;
    if (items > (1 << 30)) return fail(SF_ERR_SHAPE, "sparse_gqa(bf16): too many work items");
    ProfScope prof(SF_KERNEL_ATTEND, st);
    hipLaunchKernelGGL(kern, dim3((unsigned)align_up(items, 8)), dim3(NW * 64), lds, st, (const h16 *)a.Q, a.sq, (const h16 *)a.K,
                       a.sk, (const h16 *)vt, svt, a.head_group, a.hg_stride, a.pattern_id, a.key_valid, sel, selH, a.nH, a.nG,
                       nqb, (int)items, a.L, pl.Lp, a.U, (h16 *)a.O, a.ldo, a.row0);
    return SF_OK;
}

int32_t attend_bf16(const AttnArgs &a, const AttnPlan &pl, const void *vt, sf_strides svt,
                    const int32_t *sel, int selH, hipStream_t st)
{
    if (a.nH > 64) return fail(SF_ERR_SHAPE, "sparse_gqa(bf16): at most 64 heads");
    if (pl.staged) {
        switch (a.dh) {
        case 32: return launch_attend<32>(a, pl, vt, svt, sel, selH, st);
        case 64: return launch_attend<64>(a, pl, vt, svt, sel, selH, st);
        case 128: return launch_attend<128>(a, pl, vt, svt, sel, selH, st);
        }
    } else {
        const SliceShape s = slice_shape(a);
#define SF_SLICE(DH, QB, NW) launch_attend_slice<DH, QB, NW>(a, pl, vt, svt, sel, selH, st)
        switch (a.dh) {
        case 32: return s.qb == 2 ? SF_SLICE(32, 2, 4) : s.nw == 4 ? SF_SLICE(32, 1, 4) : SF_SLICE(32, 1, 8);
        case 64: return s.qb == 2 ? SF_SLICE(64, 2, 4) : s.nw == 4 ? SF_SLICE(64, 1, 4) : SF_SLICE(64, 1, 8);
        case 128: return s.nw == 4 ? SF_SLICE(128, 1, 4) : SF_SLICE(128, 1, 8);
        }
#undef SF_SLICE
    }
    return fail(SF_ERR_SHAPE, "sparse_gqa(bf16): dh must be 32, 64 or 128");
}

}  // namespace sf
