// An image edge as a bound on a quotient (host code, without HIP).
#pragma once

#include <cmath>
#include <cstdint>
#include <cstring>

namespace gs {

// The float after f (above it, or below), for finite f whose neighbour is finite.
inline float next_float(float f, bool above)
{
    int32_t k;
    memcpy(&k, &f, 4);
    if (k < 0) k = INT32_MIN - k;        // its place in the floats' order, both zeros at 0
    k += above ? 1 : -1;
    if (k < 0) k = INT32_MIN - k;
    memcpy(&f, &k, 4);
    return f;
}

// The least q with RN(q + centre) >= 0 and the greatest with
// RN(q + centre) <= size, FP32, for |centre| and size below 2^59, size >= 0.
//
// A sum of two floats is a multiple of the smallest subnormal, so it rounds to
// zero only if it is zero: the least q is -centre itself.  RN(q + centre) <=
// size holds up to the middle between size and the next float, less centre;
// that difference rounded (from double) is within two floats of the greatest
// q, and one to three sums find it.  24 ns for both edges, against 870 ns when
// each was found by halving the range of the floats: a call has two pairs per
// view, which the host finds before it launches.
inline void edge_interval(float centre, float size, float* lo, float* hi)
{
    *lo = 0.0f - centre;
    const double middle = 0.5 * ((double)size + (double)next_float(size, true));
    float q = (float)(middle - (double)centre);
    auto inside = [&](float x) {
        const volatile float u = x + centre;
        return u <= size;
    };
    while (!inside(q)) q = next_float(q, false);
    for (float above = next_float(q, true); inside(above); above = next_float(q, true)) q = above;
    *hi = q;
}

}  // namespace gs
