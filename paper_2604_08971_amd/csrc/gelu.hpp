// GELU of the 16-bit kernels, apart from them so that a host program can measure it.
#pragma once

#include <cmath>

#ifdef __HIPCC__
#define SF_GELU __host__ __device__ __forceinline__
#else
#define SF_GELU inline
#endif

namespace sf {

// erf-GELU z * Phi(z) for outputs that are rounded to 16 bits or fewer.  With a = |z| and s = z^2,
//     a < 1.25:  Phi(z)  = 0.5 + z R(s),                        R of degree 5 (error below 2e-8 of Phi),
//     else:      Phi(-a) = 2^(-s log2(e) / 2) * P(t),  t = 1 / (1 + 0.25 a),
// P the degree-5 polynomial that approximates erfcx(a / sqrt(2)) / 2 up to a = 15 (relative error 7e-8 up to a = 1.5, 1e-6 at
// 3, 4e-5 at 12; both by iteratively reweighted least squares).  Where Phi is small the first form loses what
// 0.5 z (1 + erf(z / sqrt(2))) loses, so it ends where the second is better; that one has no sum at all for negative z.
// Largest relative error in fp32, erff / this, 4 million values a range: -4 to -3 4.7e-4 / 3.8e-6, -2 to -1.75
// 1.2e-6 / 6.4e-7, -1.5 to -1.25 6.9e-7 / 5.3e-7, -1 to -0.8 2.7e-7 / 2.0e-7, -0.1 to 0.1 1.2e-7 / 1.2e-7, 1.25 to 1.5
// 1.4e-7 / 1.2e-7.
// About 30 instructions without a branch where erff is two divergent branches of about 20 each.  37 777 x 960 outputs with
// K 384 / 65 536 x 2176 with K 768: 86 / 330 us with erff (and the kernels of that time), 60 / 302 with the second form alone,
// whose longer polynomial and sum 1 - Phi(-a) err by 4.5e-7 around 0, 64 / 315 now; ReLU 46 / 208.
// `rcp` and `exp2` are the hardware's (1 unit in the last place each).
template <class Rcp, class Exp2>
SF_GELU float gelu_erf(float z, Rcp rcp, Exp2 exp2)
{
    const float a = fabsf(z), s = z * z;
    float r = -6.4724236e-06f;
    r = fmaf(r, s, 0.000109555076f);
    r = fmaf(r, s, -0.0011814368f);
    r = fmaf(r, s, 0.009970566f);
    r = fmaf(r, s, -0.0664897f);
    r = fmaf(r, s, 0.39894223f);
    const float t = rcp(fmaf(0.25f, a, 1.0f));
    float p = 0.2641615f;
    p = fmaf(p, t, -0.16338451f);
    p = fmaf(p, t, 0.24011181f);
    p = fmaf(p, t, 0.05214696f);
    p = fmaf(p, t, 0.10770832f);
    p = fmaf(p, t, -0.00053747342f);
    const float q = p * exp2(s * -0.72134752f);          // Phi(-a)
    const float near = fmaf(z, r, 0.5f), far = z < 0.f ? q : 1.0f - q;
    return z * (__builtin_unpredictable(a < 1.25f) ? near : far);          // a select: both sides are cheaper than a branch
}

}  // namespace sf
