// Shared host/device helpers of the gfx950 library (not used by the CPU oracle).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdarg.h>

#include "gelu.hpp"
#include "sentryfuse.h"

namespace sf {

// ---- error reporting -------------------------------------------------------
char *err_buf();                       // thread-local, 512 bytes
int32_t fail(int32_t code, const char *fmt, ...);
int32_t check_launch(const char *what);   // wraps hipGetLastError()

// ---- optional per-kernel timing (measurement aid, off by default) -----------
// While a kernel class is being profiled, every launch of that class is
// bracketed by a pair of HIP events on the launch stream.
struct ProfScope {
    ProfScope(int kernel_class, hipStream_t st);
    ~ProfScope();
    int slot;
    hipStream_t st;
};

// ---- descriptor ------------------------------------------------------------
struct Dims {
    int B, L, d, Hq, Hk, dh, F, nl, P, dtype, act, U, ffn_pad, n_sample;
    unsigned flags;
    float eps;
};
// Validates the descriptor; returns SF_OK and fills `out`.
int32_t read_desc(const sf_desc *desc, Dims &out);

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline size_t elem_size(int dtype) { return dtype == SF_BF16 ? 2 : 4; }

// Bump allocator over the caller's workspace.
struct Carver {
    char *base;
    size_t off = 0;
    explicit Carver(void *p) : base(static_cast<char *>(p)) {}
    template <class T> T *take(size_t n) {
        size_t o = off;
        off = align_up(off + n * sizeof(T), 256);
        return base ? reinterpret_cast<T *>(base + o) : nullptr;
    }
};

// ---- device helpers ----------------------------------------------------------
// The 16-bit storage and matrix-core type of this build of the library: bfloat16 (libsentryfuse.so, dtype SF_BF16)
// or, compiled with -DSF_HALF_F16, IEEE binary16 (libsentryfuse_f16.so, dtype SF_F16) - the same kernels and entry
// points; both convert from fp32 with round-to-nearest-even and accumulate in fp32.
#ifdef SF_HALF_F16
typedef _Float16 h16;
#define SF_MFMA16 __builtin_amdgcn_mfma_f32_32x32x16_f16
#define SF_FDOT2 __builtin_amdgcn_fdot2
#define SF_DTYPE_16 SF_F16
#define SF_DTYPE_16_OTHER SF_BF16
#else
typedef __bf16 h16;
#define SF_MFMA16 __builtin_amdgcn_mfma_f32_32x32x16_bf16
#define SF_FDOT2 __builtin_amdgcn_fdot2_f32_bf16
#define SF_DTYPE_16 SF_BF16
#define SF_DTYPE_16_OTHER SF_F16
#endif
typedef __attribute__((ext_vector_type(8))) h16 h16x8;
typedef __attribute__((ext_vector_type(4))) h16 h16x4;
typedef __attribute__((ext_vector_type(2))) h16 h16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(h16 x) { return (float)x; }
template <class T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ h16 from_f32<h16>(float x) { return (h16)x; }   // RNE

// Two fp32 values -> two 16-bit values in one register (a in the low half), round to nearest even.  As a vector conversion:
// one v_cvt_pk_bf16_f32, where element by element the compiler merges two results with a byte permute.  Not as inline
// assembly, in which the compiler does not see the write: it then left one instruction between the conversion and a matrix
// instruction that reads the register, where the hardware wants two, and the products were NaN.
__device__ __forceinline__ uint32_t pack2_h16(float a, float b)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, h16x2));
}

__device__ __forceinline__ float gelu_erf(float z)
{
    return gelu_erf(z, [](float x) { return __builtin_amdgcn_rcpf(x); }, [](float x) { return __builtin_amdgcn_exp2f(x); });
}

// A barrier that orders LDS only: __syncthreads() also waits for every load from memory in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// x of lane ^ O summed with the lane's own: between halves and rows of 16 by a swap, inside a row as a rotation or a permutation of four
// lanes (vector instructions; through LDS an exchange takes over 100 clocks, and a row's mean and deviations are twelve in a chain).
// O 4 only where lanes ^ 8 hold the same.
template <int O>
__device__ __forceinline__ float pair_sum(float x)
{
    if constexpr (O == 32 || O == 16) {
        const auto r = O == 32 ? __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false)
                               : __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
        constexpr int ctrl = O == 8 ? 0x128 : O == 4 ? 0x124 : O == 2 ? 0x4e : 0xb1;      // row_ror:8, row_ror:4, quad_perm
        return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xf, 0xf, false));
    }
}
// Sum over the lanes of a wave, in each of them
__device__ __forceinline__ float wave_sum(float x)
{
    return pair_sum<1>(pair_sum<2>(pair_sum<4>(pair_sum<8>(pair_sum<16>(pair_sum<32>(x))))));
}

// The first four squares of a row's deviations, in the order that every sum of them begins with (one product rounded by itself)
__device__ __forceinline__ float squares4(const float *t)
{
    return __builtin_fmaf(t[3], t[3], __builtin_fmaf(t[2], t[2], __builtin_fmaf(t[0], t[0], t[1] * t[1])));
}

// n * g + b in 16 bits.  binary16: layernorm_vec_kernel is compiled to the product that rounds to 16 bits itself; an fp32 product and
// a conversion, which the compiler may take elsewhere, differ from it in a last place now and then.  The wait is for a vector
// instruction that reads the register next: the compiler does not see that its halves are written one at a time.
__device__ __forceinline__ h16x4 scale_shift(const float *n, h16x4 g, h16x4 b)
{
#ifdef SF_HALF_F16
    const uint2 gu = __builtin_bit_cast(uint2, g), bu = __builtin_bit_cast(uint2, b);
    uint2 o;
#define SF_MIX2(D, N0, N1, G, B)                                                                                     \
    asm("v_fma_mixlo_f16 %0, %1, %3, %4 op_sel_hi:[0,1,1]\n\tv_fma_mixhi_f16 %0, %2, %3, %4 op_sel:[0,1,1] op_sel_hi:[0,1,1]\n\ts_nop 0" \
        : "=&v"(D) : "v"(N0), "v"(N1), "v"(G), "v"(B))
    SF_MIX2(o.x, n[0], n[1], gu.x, bu.x);
    SF_MIX2(o.y, n[2], n[3], gu.y, bu.y);
#undef SF_MIX2
    return __builtin_bit_cast(h16x4, o);
#else
    h16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (h16)(n[e] * (float)g[e] + (float)b[e]);
    return o;
#endif
}

// Order-preserving map of fp32 to uint32 (larger float <=> larger key).
__device__ __forceinline__ uint32_t sortable_key(float f)
{
    uint32_t u = __float_as_uint(f + 0.0f);      // -0 and +0 compare equal, as floats do
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

}  // namespace sf
