// A finite range of values cut into equal steps, for the histograms of topk.hpp and gate.hip; apart from them so that a host
// program can run it.
#pragma once

#ifdef __HIPCC__
#define SF_STEPS __host__ __device__ __forceinline__
#else
#define SF_STEPS inline
#endif

namespace sf {

// The steps per unit of n steps over [lo, hi]; false where that is no range to be cut: NaN, an infinity, one value, or one so
// narrow that the factor would leave fp32.
SF_STEPS bool cut_range(float lo, float hi, int n, float &per_unit)
{
    const float span = hi - lo;
    if (!(span > 1.0e-30f && span < 3.0e38f)) return false;
    per_unit = ((float)n - 0.5f) / span;
    return true;
}

// The step of a value of the range: the difference and the product both keep the order
SF_STEPS int step_of(float v, float lo, float per_unit, int n)
{
    const int s = (int)((v - lo) * per_unit);
    return s < n - 1 ? s : n - 1;
}

}  // namespace sf
