// Backward (paper Algorithm 2): dispatch over the kernels for small windows (fwa_backward_coop.hip), large ones
// (fwa_backward_large.hip) and wide heads (fwa_backward_wide.hip), and the reduction of the dBias partial sums that
// all of them share.
#include "fwa_device.h"
#include "fwa_internal.h"

namespace fwa {
namespace {

// dbias[h][i][j] = sum over slots of the partial sums, which the backward kernels leave in
// register order: per slot and head, block (qb, jb) holds 64 float4, the one of lane (g, n)
// carrying elements (i, j) = (16 qb + n, 16 jb + 4 g + r), r = 0..3.  A workgroup of 16 x 16
// threads owns 16 consecutive float4 of that array; thread row y adds slots y, y+16, ... in
// index order (contiguous 256-byte reads), then the 16 row sums are added in row order: a
// fixed summation tree, hence bit-reproducible.
// The grid is (quads of lanes of a row of blocks, rows of blocks, heads), so no place has to be divided into its parts: a workgroup lives
// for a trip or two to memory (24 heads of 256 tokens, 6 slots 14.2 us; 23.5 with three divisions of 32 bits in front of the loads, 20.3
// with them behind and all that lies beyond L read too).
constexpr int kReduceRows = 16;
__global__ void __launch_bounds__(16 * kReduceRows)
dbias_reduce_kernel(const f32x4* __restrict__ partial, float* __restrict__ dbias, int slots, int heads, int L,
                    int key_on_lane) {
    __shared__ f32x4 part[kReduceRows][16];
    const int x = threadIdx.x & 15, y = threadIdx.x >> 4;
    const int nb = (int)gridDim.y;
    const int b1 = (int)blockIdx.x >> 2, quad = (int)blockIdx.x & 3, b0 = (int)blockIdx.y, h = (int)blockIdx.z;
    const size_t padded = (size_t)heads * nb * nb * 64;  // float4 per slot
    const size_t f = (((size_t)h * nb + b0) * nb + b1) * 64 + 16 * quad + x;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    // Lanes and quads of lanes beyond L hold nothing (the kernels may leave them unwritten): at L = 49, where they are 38 % of the
    // array, they are neither written nor read.
    if (16 * b1 + 4 * quad >= L) return;  // the whole workgroup
    if (16 * b0 + x >= L) slots = 0;
    // 8 loads in flight per thread (one at a time leaves the kernel waiting on L2 latency); the
    // additions keep the index order
    for (int s = y; s < slots; s += 8 * kReduceRows) {
        f32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int su = s + u * kReduceRows;
            v[u] = su < slots ? partial[(size_t)su * padded + f] : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s + u * kReduceRows < slots) acc += v[u];
    }
    part[y][x] = acc;
    __syncthreads();
    if (y == 0) {
        f32x4 total = part[0][x];
#pragma unroll
        for (int r = 1; r < kReduceRows; ++r) total += part[r][x];
        if (!key_on_lane) {
            // blocks [qb][jb]; lane (g, n) holds query 16 qb + n, keys 16 jb + 4g + r
            const int i = 16 * b0 + x, j = 16 * b1 + 4 * quad;
            if (i < L) {
                float* row = dbias + ((size_t)h * L + i) * L;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (j + r < L) row[j + r] = total[r];
            }
        } else {
            // blocks [jb][qb]; lane (g, n) holds key 16 jb + n, queries 16 qb + 4g + r
            const int j = 16 * b0 + x, i = 16 * b1 + 4 * quad;
            if (j < L) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (i + r < L) dbias[((size_t)h * L + i + r) * L + j] = total[r];
            }
        }
    }
}

}  // namespace

// Workgroups along the window axis of the cooperative kernel (= dBias slots), N > 0.  Where no multiple of the mask
// period nW fits the chip the kernel forms or fetches the mask of each window and has no period to keep to.
int backward_slots(long long N, int heads, int nW, int L, bool mask, bool labels, bool dbias) {
    const int c = coop_slots(N, heads, nW);
    if (c > 0 || !(mask || labels)) return c > 0 ? c : 1;  // 1: more head groups than the chip holds workgroups
    const int most = backward_max_slots(N, heads), G = coop_window_slots(N, heads, L, mask, dbias);
    return G < most ? G : most;
}

// Upper bound of the above over all periods and forms, which the workspace query states: eight waves per CU in groups of
// four heads, or the largest count with a period, and for every call at least what any kernel needs.
int backward_max_slots(long long N, int heads) {
    const int hpb = heads < kWavesPerBlock ? heads : kWavesPerBlock;
    const int groups = (heads + hpb - 1) / hpb;
    long long slots = (cu_count() * 8 / hpb + groups - 1) / groups;
    if (slots > N) slots = N;
    if (slots < 1) slots = 1;
    const int a = coop_slots(N, heads, 1);  // period 1 gives the largest count
    return a > (int)slots ? a : (int)slots;
}

// The kernels for wide heads and for large windows add their partial sums up themselves.
hipError_t launch_backward_bf16(const BwdArgs& a, hipStream_t s) {
    if (a.C / a.heads != kHeadDim) return launch_backward_bf16_wide(a, s);
    if (a.L > kMaxBackwardL) return launch_backward_bf16_large(a, s);
    const hipError_t e = launch_backward_bf16_coop(a, s);
    if (e != hipSuccess || a.dbias == nullptr) return e;
    return launch_dbias_reduce(a, s);
}

// dbias = sum over a.slots slots of the partial sums a backward kernel left in a.partial
hipError_t launch_dbias_reduce(const BwdArgs& a, hipStream_t s, bool key_on_lane) {
    const int nb = (a.L + 15) / 16;
    // heads <= 2^15: C has at most 2^20 elements
    hipLaunchKernelGGL(dbias_reduce_kernel, dim3(4u * nb, (unsigned)nb, (unsigned)a.heads), dim3(16 * kReduceRows), 0, s,
                       reinterpret_cast<const f32x4*>(a.partial), a.dbias, a.slots, a.heads, a.L, key_on_lane ? 1 : 0);
    return hipGetLastError();
}

}  // namespace fwa
