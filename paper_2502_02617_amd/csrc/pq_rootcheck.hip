/*
 * pq_rootcheck.hip -- stand-alone check of the angle counting's short square root: compares fit_root<true> with sqrtf, bit
 * for bit, for every float of its range [2^-100, 2^101] (201 binades of 2^23 numbers and the last power of two).  Prints the
 * numbers compared and the differences; exit status 1 if there is one.
 */
#include <hip/hip_runtime.h>
#include <cstdint>
#include <cstdio>
#include <cstdlib>

#include "pq_root.h"

#define CK(x) do { hipError_t e = (x); if (e != hipSuccess) { printf("HIP error %s at %d\n", hipGetErrorString(e), __LINE__); exit(2); } } while (0)

__global__ __launch_bounds__(256) void compare(uint32_t first, uint32_t last, unsigned long long *different)
{
    uint32_t n = 0;
    for (uint32_t i = first + blockIdx.x * 256u + threadIdx.x; i <= last; i += gridDim.x * 256u) {
        const float x = __uint_as_float(i);
        n += __float_as_uint(fit_root<true>(x)) != __float_as_uint(fit_root<false>(x));
    }
    if (n) atomicAdd(different, (unsigned long long)n);
}

int main()
{
    const uint32_t first = (127u - 100u) << 23, last = (127u + 101u) << 23;
    unsigned long long *d = nullptr, h = 0;
    CK(hipMalloc(&d, sizeof h));
    CK(hipMemcpy(d, &h, sizeof h, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(compare, dim3(4096), dim3(256), 0, 0, first, last, d);
    CK(hipGetLastError());
    CK(hipMemcpy(&h, d, sizeof h, hipMemcpyDeviceToHost));
    CK(hipFree(d));
    printf("compared %u numbers, %llu different\n", last - first + 1u, h);
    return h != 0;
}
