// The two forms of the vertex transform side by side, for the test that compares their bits: one point per lane, n a
// multiple of the group's 256 threads.
#include "../paper_2103_07013_amd/csrc/raster_device.h"

namespace {
__global__ __launch_bounds__(256) void k_transforms(const float* __restrict__ matrix, const float* __restrict__ points, float4* __restrict__ on_matrix_cores,
                                                    float4* __restrict__ by_fmaf) {
    using namespace bps::dev;
    const int lane = (int)threadIdx.x & 63;
    const size_t k = (size_t)blockIdx.x * 256u + threadIdx.x;
    float M[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) M[i] = matrix[i];
    const float* row = matrix + 4 * (lane & 3);
    const ClipRows R{row[0], row[1], row[2], float4m{M[3], M[7], M[11], M[15]}};
    const float x = points[3 * k], y = points[3 * k + 1], z = points[3 * k + 2];
    const Clip4 a = to_clip(R, x, y, z), b = to_clip(M, x, y, z);
    on_matrix_cores[k] = make_float4(a.x, a.y, a.z, a.w);
    by_fmaf[k] = make_float4(b.x, b.y, b.z, b.w);
}
}  // namespace

extern "C" int transforms(const float* matrix, const float* points, unsigned n, float* on_matrix_cores, float* by_fmaf, void* stream) {
    if (n == 0 || n % 256u != 0u) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(k_transforms, dim3(n / 256u), dim3(256), 0, (hipStream_t)stream, matrix, points, reinterpret_cast<float4*>(on_matrix_cores),
                       reinterpret_cast<float4*>(by_fmaf));
    return (int)hipGetLastError();
}
