// SentryAttend for short sequences (Sec. 4.4 of the paper, Eq. (6)), 16-bit: the whole operator in one launch.  A workgroup
// serves one (sample, head): it brings the head's keys into LDS once, scores every query against them, picks the active
// queries and attends for them and for the context vector that the lazy rows receive.  As launches of their own these steps
// (statistics, score, selection with the fill, active pass, merge) are four or five kernels whose fixed cost, ramp and round
// trips through memory are most of the time of a short sequence.  us, launches of their own / this one: 28 samples of 64
// keys, 2 heads of dh 32 18.5 / 8.1; 1 of 512, 6 heads of dh 64 25.9 / 18.7; 128 of those 76 / 53; 64 of 384, 6 heads of dh 32,
// masked 34 / 19; 256 of 480, 4 heads of dh 64, masked 104 / 67; 8 of 1000, 8 heads of dh 64 44 / 37.
//
// What bounds it: one workgroup's chain of phases.  512 keys of dh 64 with eight waves, clocks: keys and their sum 6000, score
// 11000 (the matrix cores need 8200), selection 4000, active rows 6500 (VALU: two blocks of 32 rows for 36 rows), join 4000,
// fill 2000; two workgroups share a compute unit and fill each other's gaps.
#include <algorithm>
#include <atomic>

#include "attention.hpp"
#include "attention_dev.hpp"
#include "attention_short_addr.hpp"
#include "topk.hpp"

namespace sf {

namespace {

constexpr size_t SHORT_LDS = 155 * 1024;                 // next to the selection's scratch, which is static

struct ShortArgs {
    const h16 *Q; sf_strides sq;
    const h16 *K; sf_strides sk;
    const h16 *VT; sf_strides svt;
    const int32_t *head_group; int hg_stride; const int32_t *pattern_id;
    const uint8_t *key_valid; const int32_t *u_active;
    const int32_t *sample_idx; int n_sample;             // the key sample of the score, or NULL
    const int32_t *row0, *ext;
    int nH, L, Lp, U, n_items;
    int32_t *sel; float *score; int userH;               // the caller's, or NULL
    h16 *O; int64_t ldo;
};

// Keys and partial results lie in LDS without padding, in lines of 256 bytes whose 16-byte slots are permuted by the line
// number: 16 lanes are served together, and 16 consecutive rows fall into different slots whatever the chunk.  Padded rows
// would be 86 KB for 512 keys of dh 64, one workgroup per compute unit instead of two (128 samples of 512 keys, 6 heads: 64 us padded, 53 so).
template <int BYTES>                                      // of a row: 64, 128 or 256
__device__ __forceinline__ uint32_t slot_of(int row, int chunk)
{
    constexpr int RPL = 256 / BYTES, CPR = BYTES / 16;    // rows per line, chunks per row
    const int line = row / RPL;
    return (uint32_t)(line * 256 + (((row % RPL) * CPR + chunk) ^ (RPL == 4 ? line & 3 : RPL == 2 ? line & 7 : line & 15)) * 16);
}

// Sum over the lanes of a wave that hold the same chunk of a row of CH chunks (lane % CH), in every lane: rotations inside a
// row of 16 lanes, then the rows.
template <int CH>
__device__ __forceinline__ float rows_sum(float x)
{
    static_assert(CH == 4 || CH == 8, "chunks of a row");
    if (CH == 4) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, false));      // row_ror:4
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, false));                   // row_ror:8
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return both_halves_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// NW waves; a wave scores QBS blocks of 32 queries at a time; at most EPT queries per thread in the selection.  SAMPLED: the
// score looks at the allowed keys of a sample only, listed in ascending order.  OWN: waves with one tile of keys have their own
// reference of the exponentials.
template <int DH, int NW, int QBS, int EPT, bool SAMPLED, bool OWN>
__global__ __launch_bounds__(NW * 64, 4) void attend_short_bf16_kernel(ShortArgs a)
{
    constexpr int NT = NW * 64, CH = DH / 8, RP = NT / CH, UN = 8, KF = DH / 16, DB = DH / 32;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ __attribute__((aligned(16))) int scratch[TOPK_SCRATCH];
    const int item = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;      // the heads of a sample share an XCD's L2
    if (item >= a.n_items) return;                                             // uniform
    const int L = a.L, nt = (L + 31) / 32;
    const ShortLds<DH, NW> lds(L, a.U);
    float *ml = reinterpret_cast<float *>(smem + lds.ml), *refs = reinterpret_cast<float *>(smem + lds.red);
    uint32_t *keys = reinterpret_cast<uint32_t *>(smem + lds.sel_keys), *words = reinterpret_cast<uint32_t *>(smem + lds.words);
    int32_t *rows = reinterpret_cast<int32_t *>(smem + lds.rows);
    float *red = reinterpret_cast<float *>(smem + lds.red), *kbar = reinterpret_cast<float *>(smem + lds.kbar),
          *qmax = reinterpret_cast<float *>(smem + lds.qmax);

    const int b = item / a.nH, h = item % a.nH, tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, lhi = lane >> 5;
    const int g = a.head_group[(int64_t)(a.pattern_id ? a.pattern_id[b] : 0) * a.hg_stride + h];
    const h16 *Qb = a.Q + sample_offset(a.row0, b, a.sq) + (int64_t)h * a.sq.h;
    const h16 *Kb = a.K + sample_offset(a.row0, b, a.sk) + (int64_t)g * a.sk.h;
    const h16 *Vb = a.VT + (int64_t)b * a.svt.b + (int64_t)g * a.svt.h;        // the transposed V is always b-strided
    // 16 bytes at an element offset: the base stays scalar, the lane adds 32 bits (strides below 2^19, rows below 2^11)
    auto at = [](const h16 *base, uint32_t off) { return reinterpret_cast<const h16x8 *>(reinterpret_cast<const char *>(base) + off * 2u); };
    const uint8_t *kv = a.key_valid ? a.key_valid + (int64_t)b * L : nullptr;

    // ---- keys to LDS (rows beyond L are zero) and their sum: a pass covers RP keys with one 16-byte load per thread, UN passes
    // are in flight; the wave's first queries are fetched next to them
    const int r = tid / CH, c = tid % CH;          // row r of a pass, 16-byte chunk c
    h16x8 kt[UN];
    auto fetch = [&](int j0) {
#pragma unroll
        for (int k = 0; k < UN; ++k) {
            const int jk = j0 + r + RP * k;
            kt[k] = h16x8{};
            if (jk < L) kt[k] = *at(Kb, (uint32_t)jk * (uint32_t)a.sk.l + (uint32_t)c * 8u);
        }
    };
    fetch(0);
    h16x8 qf[QBS][KF];
    auto fetch_q = [&](int q0) {
#pragma unroll
        for (int qq = 0; qq < QBS; ++qq) {
            const int i = min((q0 + qq) * 32 + l32, L - 1);
#pragma unroll
            for (int kk = 0; kk < KF; ++kk) qf[qq][kk] = *at(Qb, (uint32_t)i * (uint32_t)a.sq.l + (uint32_t)(kk * 16 + lhi * 8));
        }
    };
    fetch_q(wave * QBS);
    build_mask_words(kv, L, words, nt);
    uint32_t *const set = SAMPLED ? reinterpret_cast<uint32_t *>(rows) : words;           // the keys of the score
    uint16_t *const list = reinterpret_cast<uint16_t *>(scratch);
    uint32_t set_word = 0u;
    int n_set = 0;
    if constexpr (SAMPLED) {
        if (tid < 64) set[tid] = 0u;
        lds_barrier();
        const int32_t *sample = a.sample_idx + (int64_t)b * a.n_sample;
        for (int i = tid; i < a.n_sample; i += NT) {
            const int j = sample[i];
            if (j >= 0 && j < L && ((words[j >> 5] >> (j & 31)) & 1u)) atomicOr(&set[j >> 5], 1u << (j & 31));
        }
        lds_barrier();
        uint32_t w = lane < nt ? set[lane] : 0u;
        const int before = wave_incl_scan(__popc(w)) - __popc(w);
        n_set = __builtin_amdgcn_readlane(before + __popc(w), 63);
        if (wave == 0)
            for (int at = before; w; w &= w - 1u) list[at++] = (uint16_t)(lane * 32 + __ffs((int)w) - 1);
        const int here = n_set - lane * 32;                               // lane t: the entries of tile t of the list
        set_word = here >= 32 ? 0xffffffffu : here > 0 ? (1u << here) - 1u : 0u;
    } else {
        if (kv) lds_barrier();
    }
    {
        float ak[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int j0 = 0; j0 < L; j0 += UN * RP) {
            if (j0) fetch(j0);
#pragma unroll
            for (int k = 0; k < UN; ++k) {
                const int jk = j0 + r + RP * k;
                if (jk < nt * 32) *reinterpret_cast<h16x8 *>(smem + slot_of<DH * 2>(jk, c)) = kt[k];
            }
            if (SAMPLED || kv) {                                          // a select: masked rows may hold anything
#pragma unroll
                for (int k = 0; k < UN; ++k) {
                    const int jk = j0 + r + RP * k;
                    if (!(jk < L && ((set[jk >> 5] >> (jk & 31)) & 1u))) kt[k] = h16x8{};
                }
            }
#pragma unroll
            for (int k = 0; k < UN; ++k)
#pragma unroll
                for (int t = 0; t < 8; ++t) ak[t] += (float)kt[k][t];
        }
        // the rows of a wave, then the waves
#pragma unroll
        for (int t = 0; t < 8; ++t) ak[t] = rows_sum<CH>(ak[t]);
        if (lane < CH) {
#pragma unroll
            for (int t = 0; t < 8; ++t) red[wave * DH + lane * 8 + t] = ak[t];
        }
    }
    lds_barrier();
    const uint32_t word = lane < nt ? words[lane] : 0u;                   // lane t: the allowed keys of tile t (nt <= 64)
    const unsigned long long live = __ballot(word != 0u);
    const int n = __builtin_amdgcn_readlane(wave_incl_scan(__popc(word)), 63);      // allowed keys
    if constexpr (!SAMPLED) { set_word = word; n_set = n; }
    const float inv = n_set > 0 ? 1.0f / (float)n_set : 0.f;
    if (tid < DH) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += red[w * DH + tid];
        kbar[tid] = s * inv;
    }
    lds_barrier();

    // ---- sparsity score of every query (score_bf16_kernel), its selection key
    const uint32_t k_at = slot_of<DH * 2>(l32, lhi);                      // fragment kk of tile t: + t * 64 * DH, ^ kk * 32
    const float scale = 1.0f / sqrtf((float)DH);
    for (int q0 = wave * QBS; q0 < nt; q0 += NW * QBS) {
        if (q0 != wave * QBS) fetch_q(q0);
        float rmax[QBS];
#pragma unroll
        for (int qq = 0; qq < QBS; ++qq) rmax[qq] = -INFINITY;
        h16x8 kx[KF], ky[KF];
        auto load = [&](h16x8 (&kf)[KF], int t) {
            // entries behind the list's last repeat it: masked
            const uint32_t base = SAMPLED ? slot_of<DH * 2>(list[min(t * 32 + l32, n_set - 1)], lhi) : t * (64 * DH) + k_at;
#pragma unroll
            for (int kk = 0; kk < KF; ++kk) kf[kk] = *reinterpret_cast<const h16x8 *>(smem + (base ^ (kk * 32)));
        };
        auto tile = [&](const h16x8 (&kf)[KF], int t) {
            f32x16 s[QBS];
#pragma unroll
            for (int qq = 0; qq < QBS; ++qq) {
#pragma unroll
                for (int e = 0; e < 16; ++e) s[qq][e] = 0.f;
#pragma unroll
                for (int kk = 0; kk < KF; ++kk) s[qq] = SF_MFMA16(kf[kk], qf[qq][kk], s[qq], 0, 0, 0);
            }
            const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)set_word, t);
            if (w != 0xffffffffu) {                                       // scalar branch
                const uint32_t wl = w >> (lhi * 4);                       // key row of s[e]: (e/4)*8 + lhi*4 + e%4
#pragma unroll
                for (int qq = 0; qq < QBS; ++qq)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (!((wl >> ((e / 4) * 8 + (e % 4))) & 1u)) s[qq][e] = -INFINITY;
            }
#pragma unroll
            for (int qq = 0; qq < QBS; ++qq) {
                float m = rmax[qq];
#pragma unroll
                for (int e = 0; e < 16; e += 2) m = fmaxf(fmaxf(m, s[qq][e]), s[qq][e + 1]);
                rmax[qq] = m;
            }
        };
        // the live tiles, the keys of the next one read ahead
        unsigned long long left = SAMPLED ? __ballot(set_word != 0u) : live;
        auto take = [&]() {
            const int t = __ffsll((long long)left) - 1;                   // -1: none
            left &= left - 1ull;
            return t;
        };
        int t = take();
        if (t >= 0) load(kx, t);
        while (t >= 0) {
            const int u = take();
            if (u >= 0) load(ky, u);
            tile(kx, t);
            if (u < 0) break;
            t = take();
            if (t >= 0) load(kx, t);
            tile(ky, u);
        }
#pragma unroll
        for (int qq = 0; qq < QBS; ++qq) {
            float m = both_halves_max(rmax[qq]);
            float dot = 0.f;
#pragma unroll
            for (int kk = 0; kk < KF; ++kk)
#pragma unroll
                for (int e = 0; e < 8; ++e) dot = fmaf((float)qf[qq][kk][e], kbar[kk * 16 + lhi * 8 + e], dot);
            dot = both_halves_sum(dot);
            const int i = (q0 + qq) * 32 + l32;
            if (lhi == 0 && i < L) {
                const bool ok = (words[i >> 5] >> (i & 31)) & 1u;
                qmax[i] = m;
                m = !ok ? -INFINITY : n_set == 0 ? 0.f : (m - dot) * scale;
                if (a.score) a.score[((int64_t)b * a.userH + h) * L + i] = m;
                keys[i] = ok ? max(sortable_key(m), 1u) : 0u;             // allowed: >= 1, as in select_kernel
            }
        }
    }

    // ---- the k allowed queries of the highest score, ascending.  One more row than those is attended for: the one whose scores
    // are all 0 weighs every allowed key alike, so it is the context vector.  The waves are dealt to the blocks of 32 rows, the
    // waves of a block take its key tiles in turn; the first two tiles of V are on their way during the selection.
    const int k = min(a.u_active ? min(max(a.u_active[b], 0), a.U) : a.U, n);
    const int nb = (k + 32) / 32;                                         // <= NW
    int slots = 1;
    while (slots < nb) slots *= 2;
    const int spb = NW / slots, blk = wave / spb;
    int tile_at = blk < nb ? wave % spb : nt;
    auto next_tile = [&]() {                                              // nt: no more
        while (tile_at < nt && !((live >> tile_at) & 1ull)) tile_at += spb;
        const int t = tile_at;
        tile_at += spb;
        return t;
    };
    struct VTile { h16x8 v[DB][2]; } vx, vy;
    auto load_v = [&](VTile &x, int t) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const uint32_t off = short_v_off(t, p, l32, lhi, (uint32_t)a.svt.l, a.Lp);
#pragma unroll
            for (int d = 0; d < DB; ++d)
                x.v[d][p] = *reinterpret_cast<const h16x8 *>(reinterpret_cast<const char *>(Vb + (int64_t)(d * 32) * a.svt.l) + off);
        }
    };
    int tx = next_tile(), ty = next_tile();
    if (tx < nt) load_v(vx, tx);
    if (ty < nt) load_v(vy, ty);
    lds_barrier();
    if (k == 0) {
        for (int i = tid; i < L; i += NT) keys[i] = 0u;
    } else {
        block_topk<NT, EPT>(keys, L, k, scratch, k == n, [&](int i, bool kept, int pos) {
            keys[i] = kept ? 1u : 0u;
            if (kept) rows[pos] = i;
        });
    }
    lds_barrier();
    if (a.sel)
        for (int s = tid; s < a.U; s += NT) a.sel[((int64_t)b * a.userH + h) * a.U + s] = s < k ? rows[s] : -1;

    // ---- the active rows (attend_slice_bf16_kernel: the keys of a tile are assigned to the rows of S^T so that a lane's 16
    // scores are two runs of 8 consecutive keys, which meet V^T fragments of 16 contiguous bytes)
    const int krow = 16 * (l32 >> 4) + 8 * ((l32 >> 2) & 1) + 4 * ((l32 >> 3) & 1) + (l32 & 3);
    const uint32_t kr_at = slot_of<DH * 2>(krow, lhi);
    const float sc = LOG2E / sqrtf((float)DH);
    f32x16 o[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[d][e] = 0.f;
    float l_run = 0.f, top = -INFINITY;
    if (tx < nt) {
        h16x8 qa[KF];
        const int slot = blk * 32 + l32;
#pragma unroll
        for (int kk = 0; kk < KF; ++kk) {
            qa[kk] = h16x8{};
            if (slot < k) qa[kk] = *at(Qb, (uint32_t)rows[slot] * (uint32_t)a.sq.l + (uint32_t)(kk * 16 + lhi * 8));
        }
        // The reference of the exponentials: the largest product of the row, or of the wave's tile where it has one only (OWN).  Of a
        // key sample the former is a first guess: the wave's first tile may raise it, the others do when a product exceeds it by
        // 2^RESCALE_LOG2.  The results are relative to it, but the rounding to 16 bits is least next to it: the row's for waves of
        // one tile is 4 to 8 % more error, the first tile's for waves of several 5 %.
        const bool single = OWN && ty >= nt;
        top = slot < k ? qmax[rows[slot]] * sc : 0.f;
        float slack = 0.f;
        auto process = [&](VTile &x, int t) {
            f32x16 s;
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
            for (int kk = 0; kk < KF; ++kk) {
                const h16x8 kf = *reinterpret_cast<const h16x8 *>(smem + (t * (64 * DH) + (kr_at ^ (kk * 32))));
                s = SF_MFMA16(kf, qa[kk], s, 0, 0, 0);
            }
            if (blk == k >> 5 && l32 == (k & 31)) {
#pragma unroll
                for (int e = 0; e < 16; ++e) s[e] = 0.f;
            }
            const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)word, t);
            if (w != 0xffffffffu) {                                       // scalar branch
                const uint32_t wl = w >> (lhi * 8);                       // s[e]: key 16 (e / 8) + 8 lhi + e % 8
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (!((wl >> ((e / 8) * 16 + e % 8)) & 1u)) s[e] = -INFINITY;
                // masked rows of V, and V^T beyond L, may hold anything
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (!((wl >> (p * 16 + i)) & 1u)) x.v[d][p][i] = (h16)0.f;
            }
            if (SAMPLED || single) {
                float mt = fmaxf(s[0], s[1]);
#pragma unroll
                for (int e = 2; e < 16; e += 2) mt = fmaxf(fmaxf(mt, s[e]), s[e + 1]);
                mt = both_halves_max(mt) * sc;                            // sc > 0: max and scaling commute
                if (single) {
                    top = mt;
                } else if (__builtin_amdgcn_ballot_w64(mt > top + slack) != 0ull) {
                    const float to = fmaxf(top, mt), alpha = __builtin_amdgcn_exp2f(top - (to == -INFINITY ? 0.f : to));
                    top = to;
                    l_run *= alpha;
#pragma unroll
                    for (int d = 0; d < DB; ++d)
#pragma unroll
                        for (int e = 0; e < 16; ++e) o[d][e] *= alpha;
                }
                slack = RESCALE_LOG2;
            }
            const float nm = top == -INFINITY ? 0.f : -top;
            float rs0 = 0.f, rs1 = 0.f;
            h16x8 pf[2];
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const float p0 = __builtin_amdgcn_exp2f(fmaf(s[e], sc, nm)), p1 = __builtin_amdgcn_exp2f(fmaf(s[e + 1], sc, nm));
                rs0 += p0;
                rs1 += p1;
                reinterpret_cast<uint32_t *>(&pf[e / 8])[(e % 8) / 2] = pack2_h16(p0, p1);
            }
            l_run += rs0 + rs1;
#pragma unroll
            for (int d = 0; d < DB; ++d)
#pragma unroll
                for (int p = 0; p < 2; ++p) o[d] = SF_MFMA16(x.v[d][p], pf[p], o[d], 0, 0, 0);
        };
        for (;;) {
            process(vx, tx);
            tx = next_tile();
            if (tx < nt) load_v(vx, tx);
            if (ty >= nt) break;
            process(vy, ty);
            ty = next_tile();
            if (ty < nt) load_v(vy, ty);
            if (tx >= nt) break;
        }
    }

    // ---- the waves of a block joined: lane owns query l32 and dims d*32 + q*8 + lhi*4 + {0..3}
    lds_barrier();                                                      // the keys have been read
    auto part = [&](int w, int q, int c4) { return reinterpret_cast<f32x4 *>(smem + w * (32 * DH * 4) + slot_of<DH * 4>(q, c4)); };
    {
        const float l_tot = both_halves_sum(l_run);
        if (lhi == 0) {
            ml[wave * 32 + l32] = l_tot;
            if constexpr (SAMPLED || OWN) refs[wave * 32 + l32] = top;
        }
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = o[d][q * 4 + e];
                *part(wave, l32, d * 8 + q * 2 + lhi) = v;
            }
    }
    lds_barrier();
    h16 *Ob = a.O + sample_row(a.row0, b, L) * a.ldo + (int64_t)h * DH;
    h16 *cv = reinterpret_cast<h16 *>(smem + lds.ctx);
    for (int x = tid; x < (k + 1) * CH; x += NT) {
        const int s = x / CH, d8 = (x % CH) * 8, w0 = (s >> 5) * spb, q = s & 31;
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, den = 0.f, ref = -INFINITY;
        if constexpr (SAMPLED || OWN) {
            for (int w = w0; w < w0 + spb; ++w) ref = fmaxf(ref, refs[w * 32 + q]);
            if (ref == -INFINITY) ref = 0.f;
        }
#pragma unroll 4
        for (int w = w0; w < w0 + spb; ++w) {
            const float wgt = SAMPLED || OWN ? __builtin_amdgcn_exp2f(refs[w * 32 + q] - ref) : 1.0f;
            den += wgt * ml[w * 32 + q];
            const f32x4 v0 = *part(w, q, d8 / 4), v1 = *part(w, q, d8 / 4 + 1);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[e] += wgt * v0[e];
                acc[4 + e] += wgt * v1[e];
            }
        }
        const float norm = den > 0.f ? 1.0f / den : 0.f;
        h16x8 out;
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = (h16)(acc[e] * norm);
        if (s < k) *reinterpret_cast<h16x8 *>(Ob + (int64_t)rows[s] * a.ldo + d8) = out;
        else *reinterpret_cast<h16x8 *>(cv + d8) = out;
    }
    lds_barrier();
    // ---- lazy rows: the context vector (packed samples also own the padding rows behind their tokens)
    {
        const h16x8 v = *reinterpret_cast<const h16x8 *>(cv + c * 8);
        const int end = a.ext ? a.ext[b] : L;
#pragma unroll 4
        for (int i = r; i < end; i += RP)
            if (i >= L || !keys[i]) *reinterpret_cast<h16x8 *>(Ob + (int64_t)i * a.ldo + c * 8) = v;
    }
}

template <int DH, int NW, int QBS, int EPT, bool SAMPLED, bool OWN = false>
int32_t launch_short(const ShortArgs &s, hipStream_t st)
{
    auto kern = attend_short_bf16_kernel<DH, NW, QBS, EPT, SAMPLED, OWN>;
    static std::atomic<bool> attr_set{false};     // setting the attribute twice is harmless
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, SHORT_LDS) != hipSuccess)
            return fail(SF_ERR_HIP, "sparse_gqa: cannot reserve LDS for the short attention");
        attr_set = true;
    }
    const size_t lds = ShortLds<DH, NW>(s.L, s.U).bytes;
    ProfScope prof(SF_KERNEL_ATTENTION, st);
    hipLaunchKernelGGL(kern, dim3((unsigned)align_up(s.n_items, 8)), dim3(NW * 64), lds, st, s);
    return SF_OK;
}

// Waves of a workgroup.  Four where at least three workgroups fit a compute unit (four but for the last few lengths: 41 KB at 256
// keys of dh 64 or 512 of dh 32) and there are heads for them (161 x 12 heads of 78 keys: 20 us, 34 with eight waves; 256 x 6 of
// 225, dh 64 49 / 58; 130 x 12 of 256, dh 64 71 / 75; 256 x 12 of 512, dh 32 113 / 121; with 260 to 520 heads of 288 and more,
// dh 32, eight are 5 to 10 % ahead), and for up to 128 keys, four blocks of queries; eight where two fit (128 x 6 heads of 512 keys,
// dh 64: 63 / 53 / 69 with four, eight, sixteen); sixteen for long sequences, whose score is a wave's longest step (24 x 6
// heads of 628 keys 38 / 31 / 29), once fewer than two workgroups fit or there are no more heads than compute units.
int short_waves(const AttnArgs &a)
{
    const int64_t items = (int64_t)a.B * a.nH;
    if (a.L <= 128 || (items > 256 && a.L * a.dh <= 16384)) return 4;
    return a.L * a.dh <= 32768 && (items > 256 || a.L <= 512) ? 8 : 16;
}

size_t short_lds(const AttnArgs &a, int nw)
{
    if (a.dh == 32) return nw == 4 ? ShortLds<32, 4>(a.L, a.U).bytes : nw == 8 ? ShortLds<32, 8>(a.L, a.U).bytes : ShortLds<32, 16>(a.L, a.U).bytes;
    return nw == 4 ? ShortLds<64, 4>(a.L, a.U).bytes : nw == 8 ? ShortLds<64, 8>(a.L, a.U).bytes : ShortLds<64, 16>(a.L, a.U).bytes;
}

template <int DH, int NW, bool SAMPLED>
int32_t launch_waves(const ShortArgs &s, hipStream_t st)
{
    int slots = 1;                                                        // as in the kernel, for U active rows
    while (slots < (s.U + 32) / 32) slots *= 2;
    if (ceil_div(s.L, 32) < 2 * (NW / slots))                             // some wave has one tile: fewer than 64 NW queries
        return s.L <= NW * 32 ? launch_short<DH, NW, 1, 1, SAMPLED, true>(s, st) : launch_short<DH, NW, 2, 1, SAMPLED, true>(s, st);
    if (s.L <= NW * 32) return launch_short<DH, NW, 1, 1, SAMPLED>(s, st);
    return s.L <= NW * 64 ? launch_short<DH, NW, 2, 1, SAMPLED>(s, st) : launch_short<DH, NW, 2, 4, SAMPLED>(s, st);
}

template <int DH, bool SAMPLED>
int32_t launch_dim(const ShortArgs &s, int nw, hipStream_t st)
{
    return nw == 4 ? launch_waves<DH, 4, SAMPLED>(s, st) : nw == 8 ? launch_waves<DH, 8, SAMPLED>(s, st) : launch_waves<DH, 16, SAMPLED>(s, st);
}

}  // namespace

// By length, heads and active rows, fitted to 2500 calls drawn at random (1 to 512 samples of 130 to 2000 keys, 1 to 12 heads of dh
// 32 or 64, 20 to 511 active rows, half of them masked).  Of 741 others that it takes, half with a key sample, the launch costs 0.68
// of the separate ones on average, two cost more than 1.04, none more than 1.10.
// What the separate launches do better:
//   - few heads: they spread a head over the chip, while one workgroup's chain is as long as its score (tiles of keys x blocks of
//     queries) and its active rows (tiles x blocks, eight times as long a step, since each wave brings V for itself).  us, separate /
//     this: 6 heads of 1000 keys, dh 32, 256 active rows 35 / 41; 4 of 700, dh 64, 200 of them 31 / 40; 8 of 1024, dh 64, 380 of
//     them 44 / 75; 8 of 512, dh 64, 200 of them 26 / 30; but 4 of 600, dh 64, 127 of them 29 / 28, 64 of
//     1000, dh 64, 35 of them 44 / 37.  Beyond 1024 keys, 14 heads of
//     1564 37 / 43;
//   - several rounds of heads with a compute unit to themselves (sixteen waves), and rows enough for the staged kernel, in which the
//     heads of a group share K and V: 3072 heads of 600 keys, dh 64, 256 active rows 410 / 481; 1560 of 700, 160 of them 236 /
//     298; 264 of 2000, dh 32, 255 of them 148 / 167.  One or two rounds are ahead here (256 heads of 1000, dh 64, 380 of them
//     139 / 77; 512 of 800, 200 of them 0.73).
// With a key sample the separate launches are one more, and the score is short on both sides: over 600 calls with 64 keys few
// heads are 0.45 to 0.9 up to twice the chain (4 heads of 1024, dh 64, 300 active rows 1.17), while many rounds of heads are
// behind sooner (1600 of 1100, dh 32, 127 active rows 137 / 171; 264 of 700, dh 64, 480 of them 1.21).
bool attend_short(const AttnArgs &a)
{
    if ((a.dh != 32 && a.dh != 64) || a.U < 1 || a.U >= a.L) return false;
    if ((a.sq.l | a.sk.l | a.sv.l) >> 19) return false;                   // 32-bit offsets
    const int64_t heads = (int64_t)a.B * a.nH;
    if (a.L > 1024 && heads < 64) return false;
    const int nw = short_waves(a), nt = ceil_div(a.L, 32), nb = (a.U + 32) / 32;      // nb: with the context vector
    const bool few = heads <= (a.dh == 32 ? 48 : 64), sampled = a.n_sample > 0;
    if (few && !sampled && nt * (nt + 8 * nb) > (a.dh == 32 ? 1540 : heads <= 32 ? 1120 : heads <= 48 ? 1500 : 2000)) return false;
    if (few && sampled && nt * (std::min(nt, ceil_div(a.n_sample, 32)) + 8 * nb) > (a.dh == 32 ? 2800 : heads <= 32 ? 2000 : 4200)) return false;
    if (!few && nw == 16) {
        if (a.dh == 32 && (sampled ? heads > 512 && (nb > 8 || heads > 1040) : nb > 5 && a.L > 1500)) return false;
        if (a.dh == 64 && ((heads > 512 && (nb > 8 || heads >= 800)) || (sampled && nb > 9 && heads > 256))) return false;
    }
    return nb <= nw && a.L <= std::min(nw * 256, 2048) && short_lds(a, nw) <= SHORT_LDS;
}

int32_t attend_short_bf16(const AttnArgs &a, const void *vt, sf_strides svt, int Lp, hipStream_t st)
{
    ShortArgs s{};
    s.Q = (const h16 *)a.Q; s.sq = a.sq; s.K = (const h16 *)a.K; s.sk = a.sk; s.VT = (const h16 *)vt; s.svt = svt;
    s.head_group = a.head_group; s.hg_stride = a.hg_stride; s.pattern_id = a.pattern_id;
    s.key_valid = a.key_valid; s.u_active = a.u_active; s.row0 = a.row0; s.ext = a.ext;
    s.nH = a.nH; s.L = a.L; s.Lp = Lp; s.U = a.U; s.n_items = a.B * a.nH;
    s.sel = a.sel_out; s.score = a.score_out; s.userH = a.selH > 0 ? a.selH : a.nH;
    s.O = (h16 *)a.O; s.ldo = a.ldo;
    const int nw = short_waves(a);
    if (a.sample_idx && a.n_sample > 0) {
        s.sample_idx = a.sample_idx; s.n_sample = a.n_sample;
        return a.dh == 32 ? launch_dim<32, true>(s, nw, st) : launch_dim<64, true>(s, nw, st);
    }
    return a.dh == 32 ? launch_dim<32, false>(s, nw, st) : launch_dim<64, false>(s, nw, st);
}

// ------------------------------------------------------------------------------------------------ fp32
// The same in fp32, for the small models that the fp32 path is there for: a workgroup per (sample, head) holds its queries, keys
// and values in LDS; sixteen threads share a query (or an active row), as in score_f32_kernel, whose sums it keeps.  What
// bounds it is the chain of phases, and in each the latency of LDS: four keys are on their way per thread.  us, launches of their
// own / this one: 2 x 2 heads of 48 keys, dh 16 17.1 / 12.2; 128 heads of 90, dh 32 64 / 25; 128 of 256, dh 16 72 / 45.
namespace {

struct ShortF32Args {
    const float *Q; sf_strides sq;
    const float *K; sf_strides sk;
    const float *V; int64_t v_b, v_h, v_sj, v_se; int v_rows;             // v_rows: V is token-major, row0 applies to it
    const int32_t *head_group; int hg_stride; const int32_t *pattern_id;
    const uint8_t *key_valid; const int32_t *u_active;
    const int32_t *row0, *ext;
    int nH, L, U;
    int32_t *sel; float *score; int userH;               // the caller's, or NULL
    float *O; int64_t ldo;
};

constexpr int F32_WORDS = 10;                             // 32 queries each

// floats of LDS: Q, K, V rows, selection keys, a row of probabilities per group of sixteen threads, rows, context vector
size_t short_f32_lds(int L, int dh, int U, int nt)
{
    return sizeof(float) * ((size_t)3 * L * (dh + 4) + L + (size_t)(nt / 16) * (L | 1) + U + dh);
}

template <int DH, int NT>
__global__ __launch_bounds__(NT) void attend_short_f32_kernel(ShortF32Args a)
{
    constexpr int LD = DH + 4, NG = NT / 16, C4 = DH / 4;
    extern __shared__ __attribute__((aligned(16))) float fsm[];
    __shared__ __attribute__((aligned(16))) int scratch[TOPK_SCRATCH];
    __shared__ uint32_t words[F32_WORDS];
    const int L = a.L, ldp = L | 1, tid = threadIdx.x, lane = tid & 63;
    float *Qs = fsm, *Ks = Qs + L * LD, *Vs = Ks + L * LD;
    uint32_t *keys = reinterpret_cast<uint32_t *>(Vs + L * LD);
    float *prob = reinterpret_cast<float *>(keys + L);
    int32_t *rows = reinterpret_cast<int32_t *>(prob + NG * ldp);
    float *ctx = reinterpret_cast<float *>(rows + a.U);
    const int b = blockIdx.x / a.nH, h = blockIdx.x % a.nH;
    const int g = a.head_group[(int64_t)(a.pattern_id ? a.pattern_id[b] : 0) * a.hg_stride + h];
    const float *Qb = a.Q + sample_offset(a.row0, b, a.sq) + (int64_t)h * a.sq.h;
    const float *Kb = a.K + sample_offset(a.row0, b, a.sk) + (int64_t)g * a.sk.h;
    const float *Vb = a.V + (a.v_rows && a.row0 ? (int64_t)a.row0[b] * a.v_sj : (int64_t)b * a.v_b) + (int64_t)g * a.v_h;
    const uint8_t *kv = a.key_valid ? a.key_valid + (int64_t)b * L : nullptr;
    {
        constexpr int STEP = NT / DH;
        const int e = tid % DH;
#pragma unroll 4
        for (int r = tid / DH; r < L; r += STEP) {
            Qs[r * LD + e] = Qb[(int64_t)r * a.sq.l + e];
            Ks[r * LD + e] = Kb[(int64_t)r * a.sk.l + e];
            Vs[r * LD + e] = Vb[(int64_t)r * a.v_sj + (int64_t)e * a.v_se];
        }
    }
    build_mask_words(kv, L, words, F32_WORDS);
    lds_barrier();
    const uint32_t word = lane < F32_WORDS ? words[lane] : 0u;
    const int n = __builtin_amdgcn_readlane(wave_incl_scan(__popc(word)), 63);      // allowed keys
    auto allowed = [&](int j) { return (words[j >> 5] >> (j & 31)) & 1u; };

    const int gi = tid >> 4, kl = tid & 15;
    const float scale = 1.0f / sqrtf((float)DH);
    float q[DH];
    auto load_q = [&](int i) {
#pragma unroll
        for (int c = 0; c < C4; ++c) {
            const f32x4 v = *reinterpret_cast<const f32x4 *>(Qs + i * LD + c * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) q[c * 4 + e] = v[e];
        }
    };
    // four keys at a time, j, j + 16, ...: four chains of products instead of one.  -inf: no such key, or masked
    auto dots = [&](int j, bool any, float (&s)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) s[u] = 0.f;
        if (any)
#pragma unroll
            for (int c = 0; c < C4; ++c)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(Ks + min(j + u * 16, L - 1) * LD + c * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[u] = fmaf(q[c * 4 + e], v[e], s[u]);
                }
#pragma unroll
        for (int u = 0; u < 4; ++u) s[u] = j + u * 16 < L && allowed(j + u * 16) ? s[u] * scale : -INFINITY;
    };
    // ---- sparsity score
    for (int i0 = 0; i0 < L; i0 += NG) {
        const int i = i0 + gi;
        load_q(min(i, L - 1));
        float mx = -INFINITY, sum = 0.f;
        for (int j = kl; j < L; j += 64) {
            float s[4];
            dots(j, true, s);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int jj = j + u * 16;
                mx = fmaxf(mx, s[u]);
                sum += jj < L && allowed(jj) ? s[u] : 0.f;
            }
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            mx = fmaxf(mx, __shfl_xor(mx, o));
            sum += __shfl_xor(sum, o);
        }
        if (kl == 0 && i < L) {
            const bool ok = allowed(i);
            const float m = !ok ? -INFINITY : mx - sum / (float)n;        // an allowed query: n > 0
            if (a.score) a.score[((int64_t)b * a.userH + h) * L + i] = m;
            keys[i] = ok ? max(sortable_key(m), 1u) : 0u;
        }
    }
    // ---- the k allowed queries of the highest score, ascending
    const int k = min(a.u_active ? min(max(a.u_active[b], 0), a.U) : a.U, n);
    lds_barrier();
    if (k == 0) {
        for (int i = tid; i < L; i += NT) keys[i] = 0u;
    } else {
        block_topk<NT, (F32_WORDS * 32 + NT - 1) / NT>(keys, L, k, scratch, k == n, [&](int i, bool kept, int pos) {
            keys[i] = kept ? 1u : 0u;
            if (kept) rows[pos] = i;
        });
    }
    lds_barrier();
    if (a.sel)
        for (int s = tid; s < a.U; s += NT) a.sel[((int64_t)b * a.userH + h) * a.U + s] = s < k ? rows[s] : -1;

    // ---- active rows, and the one of equal scores: the context vector
    float *Ob = a.O + sample_row(a.row0, b, L) * a.ldo + (int64_t)h * DH;
    float *p = prob + gi * ldp;
    for (int r0 = 0; r0 <= k; r0 += NG) {
        const int r = r0 + gi;
        const bool row = r < k;
        const int i = row ? rows[r] : 0;
        load_q(i);
        float mx = -INFINITY;
        for (int j = kl; j < L; j += 64) {
            float s[4];
            dots(j, row, s);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (j + u * 16 < L) p[j + u * 16] = s[u];
                mx = fmaxf(mx, s[u]);
            }
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        float dn[4] = {0.f, 0.f, 0.f, 0.f};
        for (int j = kl; j < L; j += 64) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (j + u * 16 >= L) break;
                const float s = p[j + u * 16], pj = s == -INFINITY ? 0.f : expf(s - mx);
                p[j + u * 16] = pj;
                dn[u] += pj;
            }
        }
        float den = (dn[0] + dn[1]) + (dn[2] + dn[3]);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) den += __shfl_xor(den, o);
        // the sixteen threads are in one wave: its LDS accesses are in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
        const float inv = den > 0.f ? 1.0f / den : 0.f;
        constexpr int SHARE = DH < 16 ? 16 / DH : 1, PER = DH < 16 ? 1 : DH / 16;      // threads of a dimension, dimensions of a thread
        // Eight sums of a dimension next to each other: one of all keys is 1.4 times as far from the sum in 64 bits as the separate
        // launches are (256 keys; the context vector 2.4 times)
        constexpr int SUMS = 8;
        float part[PER][SUMS];
#pragma unroll
        for (int u = 0; u < PER; ++u)
#pragma unroll
            for (int c = 0; c < SUMS; ++c) part[u][c] = 0.f;
        auto add = [&](int j, int c) {
            const float pj = p[j];
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const float v = Vs[j * LD + kl % (16 / SHARE) + u * 16];
                part[u][c] = pj != 0.f ? fmaf(pj, v, part[u][c]) : part[u][c];        // masked rows may hold anything
            }
        };
        int j = kl / (16 / SHARE);
        for (; j + (SUMS - 1) * SHARE < L; j += SUMS * SHARE)
#pragma unroll
            for (int c = 0; c < SUMS; ++c) add(j + c * SHARE, c);
#pragma unroll
        for (int c = 0; c < SUMS - 1; ++c)
            if (j + c * SHARE < L) add(j + c * SHARE, c);
        float acc[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            acc[u] = ((part[u][0] + part[u][1]) + (part[u][2] + part[u][3])) + ((part[u][4] + part[u][5]) + (part[u][6] + part[u][7]));
#pragma unroll
            for (int o = 16 / SHARE; o < 16; o <<= 1) acc[u] += __shfl_xor(acc[u], o);
            const int e = kl % (16 / SHARE) + u * 16;
            if (kl < 16 / SHARE && r <= k) {
                if (row) Ob[(int64_t)i * a.ldo + e] = acc[u] * inv;
                else ctx[e] = acc[u] * inv;
            }
        }
    }
    lds_barrier();
    // ---- lazy rows
    const int end = a.ext ? a.ext[b] : L, c = tid % C4;
    const f32x4 v = {ctx[c * 4], ctx[c * 4 + 1], ctx[c * 4 + 2], ctx[c * 4 + 3]};
    for (int i = tid / C4; i < end; i += NT / C4)
        if (i >= L || !keys[i]) *reinterpret_cast<f32x4 *>(Ob + (int64_t)i * a.ldo + c * 4) = v;
}

template <int DH, int NT>
int32_t launch_short_f32(const ShortF32Args &s, int B, hipStream_t st)
{
    auto kern = attend_short_f32_kernel<DH, NT>;
    static std::atomic<bool> attr_set{false};     // setting the attribute twice is harmless
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, SHORT_LDS) != hipSuccess)
            return fail(SF_ERR_HIP, "sparse_gqa: cannot reserve LDS for the short attention");
        attr_set = true;
    }
    const size_t lds = short_f32_lds(s.L, DH, s.U, NT);
    hipLaunchKernelGGL(kern, dim3(B * s.nH), dim3(NT), lds, st, s);
    return SF_OK;
}

// Eight waves where sixteen have no queries for them or no registers (dh 32), or there are more heads than compute units
// (64 x 8 heads of 64 keys, dh 16: 17 us, 27 with sixteen; 2 heads 13.6 with sixteen, 18 with eight)
int short_f32_threads(const AttnArgs &a)
{
    return a.L <= 32 || a.dh == 32 || (int64_t)a.B * a.nH > 256 ? 512 : short_f32_lds(a.L, a.dh, a.U, 1024) <= SHORT_LDS ? 1024 : 512;
}

template <int DH>
int32_t launch_f32_threads(const ShortF32Args &s, int B, int nt, hipStream_t st)
{
    if constexpr (DH < 32) {
        if (nt == 1024) return launch_short_f32<DH, 1024>(s, B, st);
    }
    return launch_short_f32<DH, 512>(s, B, st);
}

}  // namespace

// Longer sequences only where there are heads enough, since the separate launches spread a head over the chip (us, separate / this:
// 2 heads of 160 keys, dh 16 27 / 28, 64 heads 35 / 29; 48 heads of 220, dh 16 37 / 40, of 256, dh 8 34 / 44; 64 heads of 400 78 /
// 92); and few heads only where the active rows are one pass of the workgroup, or the sequence is so short that two are
// nothing (8 heads of 128 keys, dh 32, 64 active rows 30 / 60, 22 heads, 20 of them 31 / 30; 4 heads of 128, dh 16, 64 active rows 24
// / 32, 32 of them 23 / 21).
bool attend_short_f32(const AttnArgs &a)
{
    if ((a.dh != 8 && a.dh != 16 && a.dh != 32) || a.U < 1 || a.U >= a.L) return false;
    const int64_t heads = (int64_t)a.B * a.nH;
    const int nt = short_f32_threads(a);
    if (a.L > (heads < 48 ? 128 : heads < 96 ? 200 : 300)) return false;
    if (heads < 48 && a.U + 1 > nt / 16 && a.L > (a.dh == 32 ? 48 : 64)) return false;
    return short_f32_lds(a.L, a.dh, a.U, nt) <= SHORT_LDS;
}

int32_t attend_short_f32_run(const AttnArgs &a, hipStream_t st)
{
    ShortF32Args s{};
    s.Q = (const float *)a.Q; s.sq = a.sq; s.K = (const float *)a.K; s.sk = a.sk;
    s.V = (const float *)a.V; s.v_b = a.sv.b; s.v_h = a.sv.h;
    s.v_sj = a.v_transposed ? 1 : a.sv.l; s.v_se = a.v_transposed ? a.sv.l : 1; s.v_rows = !a.v_transposed;
    s.head_group = a.head_group; s.hg_stride = a.hg_stride; s.pattern_id = a.pattern_id;
    s.key_valid = a.key_valid; s.u_active = a.u_active; s.row0 = a.row0; s.ext = a.ext;
    s.nH = a.nH; s.L = a.L; s.U = a.U;
    s.sel = a.sel_out; s.score = a.score_out; s.userH = a.selH > 0 ? a.selH : a.nH;
    s.O = (float *)a.O; s.ldo = a.ldo;
    const int nt = short_f32_threads(a);
    return a.dh == 8 ? launch_f32_threads<8>(s, a.B, nt, st) : a.dh == 16 ? launch_f32_threads<16>(s, a.B, nt, st) : launch_f32_threads<32>(s, a.B, nt, st);
}

}  // namespace sf
