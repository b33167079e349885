// Which problems an XCD gets where they differ in cost, apart from the kernel so that a host program can run it.
#pragma once

#ifdef __HIPCC__
#define SF_DEAL __host__ __device__ __forceinline__
#else
#define SF_DEAL inline
#endif

namespace sf {

// The j-th problem of XCD x (0 .. 7) out of n, a multiple of 8: one of each eight in a row, and not the same one every time.
// The problems of a sample are neighbours (its groups) and every second or fourth sample may be the costly one; flipped bits
// from one eight to the next, through all eight of them, give every XCD its share whatever the number of groups.
SF_DEAL int deal(int x, int j)
{
    const int o = (j & 2) << 1 | (j & 4) >> 1;
    return j * 8 + (x ^ (j & 1 ? 7 - o : o));
}

}  // namespace sf
