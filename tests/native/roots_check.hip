// Counts the floats for which exact_roots differs from sqrtf, over ranges of bit patterns
// (test_gpu_roots.py).
#include "roots.h"

#include <stdint.h>

using namespace ulm;

// Thread t takes N patterns: from first + N t on, or with a stride, the first of every 64
// threads replaced by `odd` (a value that sends its whole wave to sqrtf) if mixed.
template <int N>
__global__ __launch_bounds__(256) void roots_check_kernel(uint64_t first, uint64_t threads, uint64_t stride,
                                                          int mixed, uint32_t odd, unsigned long long *bad)
{
    const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    float x[N], r[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint64_t at = stride ? t + i * stride : t * N + i;
        x[i] = __uint_as_float(mixed && (threadIdx.x & 63) == 0 && i == N / 2 ? odd : (uint32_t)(first + at));
    }
    exact_roots<N>(x, r);
    int n = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float want = sqrtf(x[i]);
        n += !(__float_as_uint(r[i]) == __float_as_uint(want) || (r[i] != r[i] && want != want));
    }
    if (t < threads && n) atomicAdd(bad, (unsigned long long)n);
}

// bad: device counter, added to.  Returns the launch's status.
extern "C" int roots_check(uint64_t first, uint64_t threads, uint64_t stride, int mixed, uint32_t odd,
                           unsigned long long *bad, void *stream)
{
    const uint64_t groups = (threads + 255) / 256;
    if (groups == 0 || groups > (1u << 23)) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(roots_check_kernel<8>, dim3((unsigned)groups), dim3(256), 0, (hipStream_t)stream, first,
                       threads, stride, mixed, odd, bad);
    return (int)hipGetLastError();
}
