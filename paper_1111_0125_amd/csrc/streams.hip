// Whether two streams run side by side. The runtime maps streams onto a few
// hardware queues (four), whose kernels start in order, and does not say which;
// streams created one after the other can get the same one.
#include "internal.h"

namespace stag {

// Raise `mine` and wait a bounded time for `other` (ticks of the 100 MHz clock).
static __global__ void k_meet(int* mine, const int* other, int* seen, int token, long long limit) {
    __hip_atomic_store(mine, token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const long long t0 = wall_clock64();
    int v;
    do {
        v = __hip_atomic_load(other, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } while (v != token && wall_clock64() - t0 < limit);
    *seen = v;
}

// One such kernel on a, then one on b: the first sees the second's flag only if b
// does not wait behind a. dev: four ints; token: not used with them before. On
// a device with other work the second can be late (1 ms: a resident kernel of a
// small lattice keeps its units for up to about that), and the answer is no.
hipError_t streams_meet(hipStream_t a, hipStream_t b, int* dev, int token, bool* apart) {
    constexpr long long limit = 100000;
    int seen = 0;
    hipLaunchKernelGGL(k_meet, dim3(1), dim3(1), 0, a, dev, dev + 1, dev + 2, token, limit);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_meet, dim3(1), dim3(1), 0, b, dev + 1, dev, dev + 3, token, limit);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&seen, dev + 2, sizeof(int), hipMemcpyDeviceToHost, a);
    const hipError_t ea = hipStreamSynchronize(a), eb = hipStreamSynchronize(b);
    if (e == hipSuccess) e = ea != hipSuccess ? ea : eb;
    *apart = e == hipSuccess && seen == token;
    return e;
}

}  // namespace stag
