// Square roots of several values at once, shared by the localiser and the motion
// estimation (both root every value of the planes or slices they read).
#pragma once

#include <hip/hip_runtime.h>

namespace ulm {

// Square roots of N values at once, correctly rounded as sqrtf's: the hardware
// reciprocal root and one Newton step on the root's residual, which is equal to sqrtf for
// every float from 2^-96 up (tests/test_gpu_roots.py compares all of them).  Smaller values
// (zeros among them), infinities and NaN take sqrtf itself, the whole wave's N at
// once.  6 instructions a value instead of sqrtf's 16.
template <int N>
__device__ inline void exact_roots(const float (&x)[N], float (&r)[N]) {
    float lo = x[0], hi = x[0];
    bool nan = false;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float y = __builtin_amdgcn_rsqf(x[i]);
        const float s = x[i] * y;
        r[i] = fmaf(fmaf(-s, s, x[i]), 0.5f * y, s);
        lo = fminf(lo, x[i]);
        hi = fmaxf(hi, x[i]);
        nan |= x[i] != x[i];
    }
    if (__ballot(!(lo >= 0x1p-96f && hi < INFINITY) || nan)) {
#pragma unroll
        for (int i = 0; i < N; ++i) r[i] = sqrtf(x[i]);
    }
}

}  // namespace ulm
