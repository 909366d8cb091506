// The tracker's square root and reciprocal as a kernel of their own, from the
// tracker's source, for the test of their roundings.
#include "fasttrack_kernels.hip"

__global__ void rounding_kernel(const float *x, float *root, float *reciprocal, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    root[i] = sqrt_rounded(x[i]);
    reciprocal[i] = rcp_rounded(x[i]);
}

extern "C" __attribute__((visibility("default"))) int rounding(const float *x, float *root, float *reciprocal, int n,
                                                               void *stream) {
    if (n < 1) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(rounding_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, x, root, reciprocal,
                       n);
    return (int)hipGetLastError();
}
