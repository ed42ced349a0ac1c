// Relative-position bias helpers: table [heads, (2k-1)^2] <-> bias [heads, L, L].
// Pure index work (the paper defers to Swin Transformer for the bias; this is
// that published indexing): pair (i, j) of a k x k window reads table column
// (y_i - y_j + k - 1) * (2k - 1) + (x_i - x_j + k - 1).
#include "fwa_device.h"
#include "fwa_internal.h"

namespace fwa {
namespace {

// A thread takes a column j and rows (h, i) of the bias; L <= 256 columns, rounded up to 2^cols, share a workgroup with others of their
// kind.  Divisions are multiplications (12 heads of 7 x 7 windows 2.98 us with five of 64 bits per element, 2.62 with two of 32 bits per
// row and one per element; 3 x 3 windows 1.81 and 1.96).  Rows counts the rows.
template <class Rows>
__global__ void __launch_bounds__(256)
bias_gather_kernel(const float* __restrict__ table, float* __restrict__ bias, Rows rows, int cols, FastDiv by_L, FastDiv by_k) {
    const uint32_t K = by_k.d, L = by_L.d, W = 2u * K - 1u;
    const uint32_t j = threadIdx.x & ((1u << cols) - 1u), each = 256u >> cols;
    if (j >= L) return;
    const uint32_t yj = fastdiv(j, by_k), xj = j - yj * K;
    for (Rows row = (Rows)blockIdx.x * each + (threadIdx.x >> cols); row < rows; row += (Rows)gridDim.x * each) {
        uint32_t h;
        if constexpr (sizeof(Rows) == 4) h = fastdiv(row, by_L);
        else h = (uint32_t)(row / L);
        const uint32_t i = (uint32_t)(row - (Rows)h * L), yi = fastdiv(i, by_k), xi = i - yi * K;
        bias[(size_t)row * L + j] = table[(size_t)h * W * W + (yi + K - 1u - yj) * W + (xi + K - 1u - xj)];
    }
}

// 16 lanes per table entry: they take its (k-|dy|)(k-|dx|) contributions, k <= 16: a lane a column of the overlap, FLIGHT of whose
// rows are in flight, and add their sums up in a fixed tree, so the result is bit-reproducible.  (One thread per entry walks up
// to k^2 loads one after the other, each a trip to L2: 11 us at 12 heads of 7 x 7 windows; the contributions dealt out to the lanes
// in turns, with a division for each, 3.7; this 2.8.)  What divides an entry's number into its parts is multiplied by instead: 3 x 3 windows,
// 12 heads 2.21 us with divisions.
constexpr int kScatterLanes = 16;
template <int FLIGHT>
__global__ void bias_scatter_kernel(const float* __restrict__ dbias, float* __restrict__ dtable, int heads, int k, FastDiv by_T, FastDiv by_W) {
    const int L = k * k, W = 2 * k - 1, T = W * W;
    const int lane = (int)(threadIdx.x % kScatterLanes);
    // total below 2^31, a step of at most 2^27; the lanes of an entry leave together
    const uint32_t total = (uint32_t)heads * (uint32_t)T, step = gridDim.x * (blockDim.x / kScatterLanes);
    for (uint32_t e = blockIdx.x * (blockDim.x / kScatterLanes) + threadIdx.x / kScatterLanes; e < total; e += step) {
        const int h = (int)fastdiv(e, by_T), at = (int)e - h * T;
        const int ay = (int)fastdiv((uint32_t)at, by_W), dy = ay - (k - 1), dx = at - ay * W - (k - 1);
        const int y0 = max(0, dy), x0 = max(0, dx), nx = k - abs(dx), ny = k - abs(dy);
        float acc = 0.f;
        if (lane < nx) {
            // element (y0 k + xi, (y0 - dy) k + xi - dx) of the head's tile, xi = x0 + lane; a row of the overlap further k rows and k
            // columns on
            const int xi = x0 + lane;
            const float* src = dbias + (size_t)h * L * L + (size_t)(y0 * k + xi) * L + ((y0 - dy) * k + xi - dx);
            const size_t next = (size_t)k * L + k;
            for (int y = 0; y < ny; y += FLIGHT) {
                float v[FLIGHT];
#pragma unroll
                for (int u = 0; u < FLIGHT; ++u) v[u] = y + u < ny ? src[(size_t)(y + u) * next] : 0.f;
#pragma unroll
                for (int u = 0; u < FLIGHT; ++u) acc += v[u];
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
    int cols = 0;
    while ((1LL << cols) < L) ++cols;
    const long long blocks = (rows + (256 >> cols) - 1) / (256 >> cols);
    const unsigned grid = (unsigned)(blocks < 8192 ? blocks : 8192);
    const FastDiv by_L = make_fastdiv((uint32_t)L), by_k = make_fastdiv((uint32_t)k);
    // a row beyond the last one is formed before it is found to be: at most 8192 * 256 on
    if (rows < 0x7fff0000LL) hipLaunchKernelGGL(bias_gather_kernel<uint32_t>, dim3(grid), dim3(256), 0, s, table, bias, (uint32_t)rows, cols, by_L, by_k);
    else hipLaunchKernelGGL(bias_gather_kernel<uint64_t>, dim3(grid), dim3(256), 0, s, table, bias, (uint64_t)rows, cols, by_L, by_k);
    return hipGetLastError();
}

hipError_t launch_bias_scatter(const float* dbias, float* dtable, int heads, int k, hipStream_t s) {
    // a launch holds fewer than 2^32 threads: beyond 2^27 entries the workgroups take several each
    const long long total = (long long)heads * (2 * k - 1) * (2 * k - 1);
    if (total > 0x7fffffffLL) return hipErrorInvalidValue;
    const long long per_block = 256 / kScatterLanes, blocks = (total + per_block - 1) / per_block;
    const unsigned grid = (unsigned)(blocks < (1LL << 23) ? blocks : (1LL << 23));
    const FastDiv by_T = make_fastdiv((uint32_t)((2 * k - 1) * (2 * k - 1))), by_W = make_fastdiv((uint32_t)(2 * k - 1));
    // loads for rows that the overlap does not have take their turns too: 12 heads of 4 x 4 windows 2.14 us with eight, 2.09 with four
    if (k <= 4) hipLaunchKernelGGL(bias_scatter_kernel<4>, dim3(grid), dim3(256), 0, s, dbias, dtable, heads, k, by_T, by_W);
    else hipLaunchKernelGGL(bias_scatter_kernel<8>, dim3(grid), dim3(256), 0, s, dbias, dtable, heads, k, by_T, by_W);
    return hipGetLastError();
}

}  // namespace fwa
