// Relative-position bias helpers: table [heads, (2k-1)^2] <-> bias [heads, L, L].
// Pure index work (the paper defers to Swin Transformer for the bias; this is
// that published indexing): pair (i, j) of a k x k window reads table column
// (y_i - y_j + k - 1) * (2k - 1) + (x_i - x_j + k - 1).
#include "fwa_internal.h"

namespace fwa {
namespace {

__global__ void bias_gather_kernel(const float* __restrict__ table, float* __restrict__ bias, int heads, int k) {
    const int L = k * k, T = (2 * k - 1) * (2 * k - 1);
    const long long total = (long long)heads * L * L;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const int j = (int)(e % L);
        const int i = (int)((e / L) % L);
        const int h = (int)(e / ((long long)L * L));
        const int dy = i / k - j / k + k - 1;
        const int dx = i % k - j % k + k - 1;
        bias[e] = table[(size_t)h * T + dy * (2 * k - 1) + dx];
    }
}

// 16 lanes per table entry: they take its (k-|dy|)(k-|dx|) contributions in turns and add their sums up in a fixed
// tree, so the result is bit-reproducible.  (One thread per entry walks up to k^2 loads one after the other, each a
// trip to L2: 11 us at 12 heads of 7 x 7 windows against 4 now, 60 against 5 at 4 heads of 16 x 16.)
constexpr int kScatterLanes = 16;
__global__ void bias_scatter_kernel(const float* __restrict__ dbias, float* __restrict__ dtable, int heads, int k) {
    const int L = k * k, W = 2 * k - 1, T = W * W;
    const int lane = (int)(threadIdx.x % kScatterLanes);
    // total below 2^31, a step of at most 2^27; the lanes of an entry leave together
    const uint32_t total = (uint32_t)heads * (uint32_t)T, step = gridDim.x * (blockDim.x / kScatterLanes);
    for (uint32_t e = blockIdx.x * (blockDim.x / kScatterLanes) + threadIdx.x / kScatterLanes; e < total; e += step) {
        const int h = (int)e / T, at = (int)e % T;
        const int dy = at / W - (k - 1), dx = at % W - (k - 1);
        const int y0 = max(0, dy), x0 = max(0, dx), nx = k - abs(dx), count = (k - abs(dy)) * nx;
        const float* src = dbias + (size_t)h * L * L;
        float acc = 0.f;
#pragma unroll 4
        for (int c = lane; c < count; c += kScatterLanes) {
            const int yi = y0 + c / nx, xi = x0 + c % nx;
            acc += src[(size_t)(yi * k + xi) * L + (yi - dy) * k + (xi - dx)];
        }
#pragma unroll
        for (int d = kScatterLanes / 2; d > 0; d /= 2) acc += __shfl_xor(acc, d, kScatterLanes);
        if (lane == 0) dtable[e] = acc;
    }
}

__global__ void zero_f32_kernel(float* __restrict__ dst, size_t count) {
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < count; e += (size_t)gridDim.x * blockDim.x)
        dst[e] = 0.f;
}

// bf16 -> fp32 (exact: the 16 bits become the upper half of the word)
__global__ void widen_bf16_kernel(const uint16_t* __restrict__ src, float* __restrict__ dst, size_t count) {
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < count; e += (size_t)gridDim.x * blockDim.x)
        dst[e] = __builtin_bit_cast(float, (uint32_t)src[e] << 16);
}

}  // namespace

hipError_t launch_widen_bf16(const void* src, float* dst, size_t count, hipStream_t s) {
    const size_t blocks = (count + 255) / 256;
    hipLaunchKernelGGL(widen_bf16_kernel, dim3((unsigned)(blocks > 1024 ? 1024 : blocks)), dim3(256), 0, s,
                       static_cast<const uint16_t*>(src), dst, count);
    return hipGetLastError();
}

// A fill kernel rather than a memset node, so that callers may capture it in a graph.
hipError_t launch_zero_f32(float* dst, size_t count, hipStream_t s) {
    const size_t blocks = (count + 255) / 256;
    hipLaunchKernelGGL(zero_f32_kernel, dim3((unsigned)(blocks > 1024 ? 1024 : blocks)), dim3(256), 0, s, dst, count);
    return hipGetLastError();
}

hipError_t launch_bias_gather(const float* table, float* bias, int heads, int k, hipStream_t s) {
    const long long total = (long long)heads * k * k * k * k;
    const unsigned grid = (unsigned)((total + 255) / 256 > 4096 ? 4096 : (total + 255) / 256);
    hipLaunchKernelGGL(bias_gather_kernel, dim3(grid), dim3(256), 0, s, table, bias, heads, k);
    return hipGetLastError();
}

hipError_t launch_bias_scatter(const float* dbias, float* dtable, int heads, int k, hipStream_t s) {
    // a launch holds fewer than 2^32 threads: beyond 2^27 entries the workgroups take several each
    const long long total = (long long)heads * (2 * k - 1) * (2 * k - 1);
    if (total > 0x7fffffffLL) return hipErrorInvalidValue;
    const long long per_block = 256 / kScatterLanes, blocks = (total + per_block - 1) / per_block;
    const unsigned grid = (unsigned)(blocks < (1LL << 23) ? blocks : (1LL << 23));
    hipLaunchKernelGGL(bias_scatter_kernel, dim3(grid), dim3(256), 0, s, dbias, dtable, heads, k);
    return hipGetLastError();
}

}  // namespace fwa
