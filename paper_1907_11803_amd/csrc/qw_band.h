// The FP32 error band around a query's K-th key (float rows).
#pragma once
#include "qw_internal.h"

namespace qw {

// Band threshold, rounded up to float: with keys F of |F - D| <= eps D + err,
// the K-th distance is at most (F_K + err) / (1 - eps), so every key of the
// exact top-K is at most (F_K + err) (1 + eps) / (1 - eps) + err.  Keys near
// FP32's end may stand for larger distances: no bound.
__device__ inline float band_threshold(float FK, float eps, float err)
{
    if (!(FK < 1e37f)) return INFINITY;
    const double t = ((double)FK + (double)err) * (1.0 + (double)eps) / (1.0 - (double)eps) + (double)err + 0x1p-100;
    float f = (float)t;
    if ((double)f < t) f = nextafterf(f, INFINITY);
    return f;
}

}  // namespace qw
