// Relative-position bias helpers: table [heads, (2k-1)^2] <-> bias [heads, L, L].
// Pure index work (the paper defers to Swin Transformer for the bias; this is
// that published indexing): pair (i, j) of a k x k window reads table column
// (y_i - y_j + k - 1) * (2k - 1) + (x_i - x_j + k - 1).
#include "fwa_internal.h"

namespace fwa {
namespace {

// A workgroup takes rows (h, i) of the bias, a thread columns j: what depends on the row alone is formed once, and no element costs
// more than one division of 32 bits (five of 64 bits before; 12 heads of 7 x 7 windows 2.98 -> 2.62 us).  Rows counts the rows.
template <class Rows>
__global__ void bias_gather_kernel(const float* __restrict__ table, float* __restrict__ bias, int heads, int k) {
    const uint32_t K = (uint32_t)k, L = K * K, W = 2u * K - 1u;
    const Rows rows = (Rows)heads * L;
    for (Rows row = blockIdx.x; row < rows; row += gridDim.x) {
        const uint32_t h = (uint32_t)(row / L), i = (uint32_t)(row - (Rows)h * L), yi = i / K, xi = i - yi * K;
        const float* const src = table + (size_t)h * W * W + (size_t)(yi + K - 1u) * W + (xi + K - 1u);
        float* const dst = bias + (size_t)row * L;
        for (uint32_t j = threadIdx.x; j < L; j += blockDim.x) {
            const uint32_t yj = j / K, xj = j - yj * K;
            dst[j] = *(src - (size_t)yj * W - xj);
        }
    }
}

// 16 lanes per table entry: they take its (k-|dy|)(k-|dx|) contributions, k <= 16: a lane a column of the overlap, 8 of whose rows
// are in flight, and add their sums up in a fixed tree, so the result is bit-reproducible.  (One thread per entry walks up
// to k^2 loads one after the other, each a trip to L2: 11 us at 12 heads of 7 x 7 windows; the contributions dealt out to the lanes
// in turns, with a division for each, 3.7; this 2.8.)
constexpr int kScatterLanes = 16;
__global__ void bias_scatter_kernel(const float* __restrict__ dbias, float* __restrict__ dtable, int heads, int k) {
    const int L = k * k, W = 2 * k - 1, T = W * W;
    const int lane = (int)(threadIdx.x % kScatterLanes);
    // total below 2^31, a step of at most 2^27; the lanes of an entry leave together
    const uint32_t total = (uint32_t)heads * (uint32_t)T, step = gridDim.x * (blockDim.x / kScatterLanes);
    for (uint32_t e = blockIdx.x * (blockDim.x / kScatterLanes) + threadIdx.x / kScatterLanes; e < total; e += step) {
        const int h = (int)(e / (uint32_t)T), at = (int)(e % (uint32_t)T);
        const int dy = at / W - (k - 1), dx = at % W - (k - 1);
        const int y0 = max(0, dy), x0 = max(0, dx), nx = k - abs(dx), ny = k - abs(dy);
        float acc = 0.f;
        if (lane < nx) {
            // element (y0 k + xi, (y0 - dy) k + xi - dx) of the head's tile, xi = x0 + lane; a row of the overlap further k rows and k
            // columns on
            const int xi = x0 + lane;
            const float* src = dbias + (size_t)h * L * L + (size_t)(y0 * k + xi) * L + ((y0 - dy) * k + xi - dx);
            const size_t next = (size_t)k * L + k;
            for (int y = 0; y < ny; y += 8) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = y + u < ny ? src[(size_t)(y + u) * next] : 0.f;
#pragma unroll
                for (int u = 0; u < 8; ++u) acc += v[u];
            }
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
    const long long L = (long long)k * k, rows = heads * L;
    const unsigned grid = (unsigned)(rows < 8192 ? rows : 8192), block = L <= 64 ? 64u : 256u;
    if (rows < 0x7fff0000LL) hipLaunchKernelGGL(bias_gather_kernel<uint32_t>, dim3(grid), dim3(block), 0, s, table, bias, heads, k);
    else hipLaunchKernelGGL(bias_gather_kernel<uint64_t>, dim3(grid), dim3(block), 0, s, table, bias, heads, k);
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
