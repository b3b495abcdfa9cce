// Inversion of the rounded VRAM additions (plain C++, shared by the device
// code and a CPU test).
#pragma once

#include <cfloat>
#include <cmath>

#ifdef __HIPCC__
#define MF_HD __host__ __device__
#else
#define MF_HD
#endif

namespace mfi {

// The largest float x with fl(x + v) <= thr (fl: fp32, to nearest even; v
// finite, thr finite or -inf); -inf when only -inf satisfies it.  fl(x + v)
// is monotone in x and stays at or below thr exactly up to the midpoint m of
// thr and the next float (the tie at m itself goes to the even one), so x is
// m - v rounded down, give or take the tie and the rounding of m - v in fp64
// (2^-53 relative, against a float spacing of 2^-24): one float step, which
// the additions themselves settle.
MF_HD inline float vram_inverse(float thr, float v)
{
    // the infinities stand for +-2^128, the values beyond the largest float
    const double low = thr == -INFINITY ? -0x1p128 : (double)thr;
    const double next = thr == FLT_MAX ? 0x1p128 : (double)nextafterf(thr, INFINITY);
    const double d = 0.5 * (low + next) - (double)v;
    float x;
    if (d < -(double)FLT_MAX) {
        x = -INFINITY;
    } else if (d >= 0x1p128) {
        x = FLT_MAX;
    } else {
        x = (float)d;
        if ((double)x > d) x = nextafterf(x, -INFINITY);
    }
    for (int i = 0; i < 3 && x < FLT_MAX; i++) {
        const float y = nextafterf(x, INFINITY);
        const float s = y + v;
        if (!(s <= thr)) break;
        x = y;
    }
    for (int i = 0; i < 3 && x > -INFINITY; i++) {
        const float s = x + v;
        if (s <= thr) break;
        x = nextafterf(x, -INFINITY);
    }
    return x + 0.f;   // -0 as +0
}

}  // namespace mfi
