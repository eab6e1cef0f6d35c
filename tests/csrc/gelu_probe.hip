// gelu_probe.hip -- test-only access to the network's GELU (csrc/hawkes_gelu.h): value and slope of
// n FP32 arguments, as batched inference forms them (fast = 1) and with erff and expf (fast = 0).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "hawkes_gelu.h"

__global__ __launch_bounds__(256) void k_gelu(int fast, int64_t n, const float *x, float *value, float *slope)
{
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n)
        return;
    if (fast) {
        const hawkes::Gelu g = hawkes::gelu_all(x[i]);
        value[i] = g.a;
        slope[i] = g.d1;
    } else {
        value[i] = hawkes::gelu(x[i]);
        slope[i] = hawkes::gelu_d1(x[i]);
    }
}

// Device arrays of n floats.  Returns 0, or -1 for bad arguments, -4 if the launch failed.
extern "C" int gelu_probe(int fast, int64_t n, const float *d_x, float *d_value, float *d_slope, void *stream)
{
    if (n < 1 || n > (int64_t(1) << 30) || !d_x || !d_value || !d_slope)
        return -1;
    hipLaunchKernelGGL(k_gelu, dim3(unsigned((n + 255) / 256)), dim3(256), 0, reinterpret_cast<hipStream_t>(stream), fast,
                       n, d_x, d_value, d_slope);
    return hipGetLastError() == hipSuccess ? 0 : -4;
}
