// Calibration of the smoothing factors (Eq. 4): lambda_i = sqrt(max over the calibration tokens of |K[., i]|),
// per KV head and channel.  |x| of an fp16 value is exact and a non-negative fp32 orders like its
// bit pattern, so the maximum is taken with integer atomics directly in the output array and is
// the same whatever the order; a last pass takes the square root in place.
#include "common.h"

namespace vecinfer {

namespace {

constexpr int kCalBlock = 256;
constexpr int kCalTokens = 256;     // tokens per workgroup

__global__ void lambda_zero_kernel(float *lam, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) lam[i] = 0.f;
}

// grid (token chunks, Hkv, B); a thread owns 8 adjacent channels of every kRows-th token of the chunk, one 16-byte
// load each, all in flight together (behind the last token: that one again); the kRows maxima of a channel meet in LDS, so
// that a workgroup sends one atomic per channel.  Bound by memory: 32768 x 8 tokens, D = 128 (67 MB, 11 us at the rate
// of a plain read) 38 us with a 2-byte load per thread, token and channel and two atomics per channel, 12 with this.
template <int D>
__global__ __launch_bounds__(kCalBlock) void lambda_max_kernel(const __half *k, float *lam, int Hkv, long long T)
{
    constexpr int kLanes = D / 8, kRows = kCalBlock / kLanes, kSteps = kCalTokens / kRows;
    __shared__ float max_s[kRows][D];
    const int l = threadIdx.x % kLanes, r = threadIdx.x / kLanes;
    const int g = blockIdx.y, b = blockIdx.z;
    const long long t0 = (long long)blockIdx.x * kCalTokens;
    const long long last = t0 + kCalTokens < T ? t0 + kCalTokens - 1 : T - 1;
    const __half *row = k + ((size_t)b * Hkv + g) * T * D + 8 * l;
    uint4 raw[kSteps];
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        const long long t = t0 + r + i * kRows;
        raw[i] = *reinterpret_cast<const uint4 *>(row + (t < last ? t : last) * D);
    }
    float mx[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        __half h[8];
        __builtin_memcpy(h, &raw[i], 16);
#pragma unroll
        for (int j = 0; j < 8; ++j) mx[j] = fmaxf(mx[j], fabsf(__half2float(h[j])));
    }
#pragma unroll
    for (int j = 0; j < 8; j += 4) *reinterpret_cast<float4 *>(&max_s[r][8 * l + j]) = make_float4(mx[j], mx[j + 1], mx[j + 2], mx[j + 3]);
    __syncthreads();
    if (threadIdx.x < D) {
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < kRows; ++i) m = fmaxf(m, max_s[i][threadIdx.x]);
        atomicMax(reinterpret_cast<unsigned *>(lam) + (size_t)g * D + threadIdx.x, __float_as_uint(m));
    }
}

__global__ void lambda_finalize_kernel(float *lam, int n, float floor_value)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) lam[i] = fmaxf(sqrtf(lam[i]), floor_value);
}

} // namespace

int launch_calibrate_lambda(const __half *k, float *lam, int B, int Hkv, int D, long long T, float floor_value,
                            hipStream_t stream)
{
    const int n = Hkv * D;
    hipLaunchKernelGGL(lambda_zero_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, lam, n);
    if (hipGetLastError() != hipSuccess) return -4;
    dim3 grid((unsigned)((T + kCalTokens - 1) / kCalTokens), Hkv, B);
    if (D == 128)
        hipLaunchKernelGGL(lambda_max_kernel<128>, grid, dim3(kCalBlock), 0, stream, k, lam, Hkv, T);
    else
        hipLaunchKernelGGL(lambda_max_kernel<64>, grid, dim3(kCalBlock), 0, stream, k, lam, Hkv, T);
    if (hipGetLastError() != hipSuccess) return -4;
    hipLaunchKernelGGL(lambda_finalize_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, lam, n, floor_value);
    return hipGetLastError() == hipSuccess ? 0 : -4;
}

} // namespace vecinfer
