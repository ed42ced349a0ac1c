// fp32 forward for windows of more than 64 tokens, head width 32.
//
// The fp32 matrix instruction does 32 products a cycle and SIMD, the bf16 one 512.  An fp32 value is the sum of three bf16
// values (8 + 8 + 8 significant bits), and a product of two such sums is, but for terms below 2^-26 of it, six bf16
// products, each exact and summed in fp32: x y = h h' + (h m' + m h') + (h l' + m m' + l h').  So the same result to the
// last bits of fp32 costs 6 products of the 16 times as fast kind (the kernel before this one waited for the fp32 instruction in half
// of its cycles).  What that needs: every K, V and Q value is split once per tile, every probability once, 3.5 vector
// instructions each, or 1.5 and half a matrix instruction (split3).  The error against 64 bits is smaller than that of the fp32 instruction, whose sums are rounded after
// every four products instead of 32: 1.2e-7 .. 1.7e-7 (2-norm) against 2.4e-7 .. 3.7e-7 over 81 to 256 tokens.
//
// A workgroup holds K and V of a (window, head) tile in LDS as three bf16 slabs each and walks the tiles t, t + grid, ...;
// the next tile's rows are on their way into registers meanwhile.  W waves share the 16-query blocks of the tile.  "Query on
// the lane": lane (g, n) has query 16 qb + n and in key block jb the keys 4g .. 4g + 3 in fp32, all scores of the block in
// registers; softmax and additive term are fp32 as before.  The term is fetched per tile, four key blocks at a time and
// four ahead of the products that it is added to (in front of the same four: 95 us instead of 75 below; through LDS in whole lines:
// 84).
//
// Values that do not fit (Q and K from 2^60 on, V from 2^86, infinities, NaN) are looked for on the way, and the tiles (K, V) or
// query blocks (Q) that have some go through the fp32 matrix instruction, with K from memory and V in LDS as it is: 146 us
// where all tiles do in the first case below (96 the kernel before this one), 60 at 256 tiles of 12 x 12, 4 heads (47), 41 at 864 of
// 9 x 9, 2 heads (37).
//
// Measured, 256 windows of 16 x 16 tokens, 4 heads, bias: 99 -> 76 us (62: the fp32 instruction's own time), 73.5 since
// the remainders of the splits come from the matrix core (1056 tiles of 14 x 14 68.6 -> 65.8, 4096 of 12 x 12 without a term
// 87.4 -> 82.2); 264 tiles of 14 x 14 41 -> 25; 64 windows of 12 x 12, 3 heads 12.5 -> 10.  A wave spends its time in thirds on scores, on probabilities and their
// products, and on stores, splits and barriers, which two or three waves per SIMD overlap in part: in the first case the
// vector ALU is busy for 32 % of the cycles, the matrix cores for 32 %, the LDS for 24 %.
#include "fwa_device.h"
#include "fwa_internal.h"
#include "fwa_softmax.h"
#include "fwa_split3.h"

#include <algorithm>

namespace fwa {
namespace {

// Waves per workgroup.  LDS and registers leave a CU room for 8 waves (12 while the kernel fits 168 registers: up to 7 blocks,
// 8 without an additive term), and what counts is that they come as two workgroups or more, one loading and splitting while the
// other computes, with few idle turns (NB / (W ceil(NB / W))).  W = 3 up to 6 blocks (1728 tiles of 81 tokens 37.0 us with
// 6 waves, 27.5 with 3), 4 up to 13 (1536 of 169: 83.1 with 6, 66 with 4; 264 of 196 27.5 with 7, 25.3 with 4).  From 14 blocks
// on, and at 9 without an additive term, one workgroup has the CU to itself and takes as many waves as fit; at 9 with one,
// 9 waves would have to share the registers of 12 and spill (1584 tiles 78.0, 74.4 with 5).
constexpr int f32_rows_waves(int nb, bool bm) {
    return nb <= 6 ? 3 : (nb == 9 ? (bm ? 5 : 9) : (nb <= 13 ? 4 : (nb <= 14 ? 7 : 8)));
}
// Magnitudes below which the sums of 32 score products, resp. of 256 products of weights and V, both lifted, stay finite in every
// part (see fits_lifted)
constexpr float kMostQK = 0x1p60f, kMostV = 0x1p86f;
constexpr uint32_t kRowV = 144;  // bytes from row to row of a V that is not split (32 floats and room between the banks)
template <int NB>
constexpr size_t f32_rows_lds() { return (size_t)6 * 16 * NB * 64 + 16; }

// Splits with the remainders from the matrix core -- but not with an additive term at up to 7 blocks, where 168 registers would spill more
// (2304 tiles of 10 x 10 tokens 45.0 -> 46.8 us; of 9 x 9 3456 tiles 48.5 -> 47.2 but 48 tiles 5.38 -> 5.63), and at 9 (2048 tiles of
// 12 x 12 even, 48 tiles 7.03 -> 7.20).
constexpr bool f32_rows_matrix(int nb, bool bm, int w) { return !(bm && w < nb && (nb <= 7 || nb == 9)); }

template <int NB, bool BM, int W, bool MATRIX>
__global__ void __launch_bounds__(64 * W, W < NB && (NB <= 7 || (NB == 8 && !BM)) ? 3 : 2) fwd_f32_rows_kernel(FwdArgs p, uint32_t parts, uint32_t tiles) {
    constexpr int ROWS = 16 * NB;
    constexpr int PASSES = (ROWS + 8 * W - 1) / (8 * W);  // the workgroup moves 8 W slab rows per pass
    constexpr uint32_t SLAB = ROWS * 64;                  // bytes of a plane; rows of 32 bf16
    constexpr int NB2 = (NB + 1) / 2;
    extern __shared__ __attribute__((aligned(16))) char ldsb[];  // K planes h, m, l; V planes; two flags
    const int tid = threadIdx.x, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = p.L;
    const uint32_t row_bytes = (uint32_t)p.ldq * 4u, row_out = (uint32_t)p.ldo * 4u;
    const uint32_t tile_bytes = (uint32_t)(L - 1) * row_bytes + 4u * kHeadDim;
    char* const lk = ldsb;
    char* const lv = ldsb + 3 * SLAB;
    int* const flag = reinterpret_cast<int*>(ldsb + 6 * SLAB);
    const uint32_t srow = (uint32_t)tid >> 3, scol = (uint32_t)tid & 7u;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    // MATRIX: splits with the remainders from the matrix core, those of the next pair's weights beside the products of this one
    const bf16x4 minus_one = minus_identity(g, n);
    auto split = [&](const f32x4& x) {
        if constexpr (MATRIX) return split3(minus_one, x);
        else return split3(x);
    };

    auto tile_of = [&](uint32_t t, uint32_t& w, uint32_t& h) {
        const uint32_t bh = t / parts;
        w = bh / (uint32_t)p.heads, h = bh - w * (uint32_t)p.heads;
    };
    f32x4 nk[PASSES], nv[PASSES], nqa = zero, nqc = zero;  // K and V rows of the next tile, the wave's first Q rows of it
    auto request = [&](uint32_t t) {
        uint32_t w, h;
        tile_of(t, w, h);
        const size_t tile = ((size_t)w * L * p.ldq + (size_t)h * kHeadDim) * 4u;
        const __amdgpu_buffer_rsrc_t rk = make_rsrc((const char*)p.k + tile, tile_bytes);
        const __amdgpu_buffer_rsrc_t rv = make_rsrc((const char*)p.v + tile, tile_bytes);
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {  // rows beyond L arrive as zeros
            const uint32_t off = (8 * W * i + srow) * row_bytes + scol * 16u;
            nk[i] = load_f32x4(rk, off);
            nv[i] = load_f32x4(rv, off);
        }
        const __amdgpu_buffer_rsrc_t rq = make_rsrc((const char*)p.q + tile, tile_bytes);
        const uint32_t off_q = (uint32_t)(16 * (t % parts + parts * wave) + n) * row_bytes + 32u * g;
        nqa = load_f32x4(rq, off_q);  // channels 8g .. 8g + 7
        nqc = load_f32x4(rq, off_q + 16u);
    };
    auto put = [&](char* slab, uint32_t row, const f32x4& x) {
        const Planes s = split(x);
        char* const to = slab + row * 64u + scol * 8u;
        *reinterpret_cast<u32x2*>(to) = s.h;
        *reinterpret_cast<u32x2*>(to + SLAB) = s.m;
        *reinterpret_cast<u32x2*>(to + 2 * SLAB) = s.l;
    };
    if (tid < 2) flag[tid] = 0;
    request(blockIdx.x);
    __syncthreads();

    uint32_t turn = 0u;
    for (uint32_t t = blockIdx.x; t < tiles; t += gridDim.x, turn ^= 1u) {
        float top = 0.f, top_v = 0.f;
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const uint32_t row = 8 * W * i + srow;
            top = largest(top, nk[i]);
            top_v = largest(top_v, nv[i]);
            if (ROWS % (8 * W) == 0 || row < (uint32_t)ROWS) {
                put(lk, row, nk[i]);
                put(lv, row, nv[i] * kLift);
            }
        }
        // K and Q go without the lift: what they lose, 2^-134 of a value below 2^-110, is nothing to a score, whatever Q and K
        // that fit it is multiplied by, unless the scale makes it something.
        if (__any(!(top < kMostQK) || !(top_v < kMostV)) || !(fabsf(p.scale) < 0x1p40f)) flag[turn] = 1;
        __syncthreads();
        const bool wide = __builtin_amdgcn_readfirstlane(flag[turn]) != 0;
        if (wide) {  // V as it is, over its planes
            uint32_t w, h;
            tile_of(t, w, h);
            const __amdgpu_buffer_rsrc_t rv = make_rsrc((const char*)p.v + ((size_t)w * L * p.ldq + (size_t)h * kHeadDim) * 4u, tile_bytes);
#pragma unroll 1
            for (uint32_t row = srow; row < (uint32_t)ROWS; row += 8 * W)
                *reinterpret_cast<f32x4*>(lv + row * kRowV + scol * 16u) = load_f32x4(rv, row * row_bytes + scol * 16u);
            __syncthreads();
        }
        if (tid == 0) flag[turn ^ 1u] = 0;  // read by all before the barrier that ended the last tile
        f32x4 qa = nqa, qc = nqc;
        if (t + gridDim.x < tiles) request(t + gridDim.x);

        uint32_t w, h;
        tile_of(t, w, h);
        const size_t tile = ((size_t)w * L * p.ldq + (size_t)h * kHeadDim) * 4u;
        const __amdgpu_buffer_rsrc_t rq = make_rsrc((const char*)p.q + tile, tile_bytes);
        const __amdgpu_buffer_rsrc_t ro =
            make_rsrc((char*)p.o + ((size_t)w * L * p.ldo + (size_t)h * kHeadDim) * 4u, (uint32_t)(L - 1) * row_out + 4u * kHeadDim);
        BiasSrc rb = no_bias();
        MaskSrc msk = {make_rsrc(nullptr, 0), 0.f, false};
        const bool has_msk = BM && (p.mask || p.labels);
        if (BM) {
            rb = bias_of_head(p, h);
            msk = mask_of_window(p, w);
        }
        for (int qb = (int)(t % parts + parts * wave); qb < NB; qb += (int)parts * W) {
            const bool fp32 = wide || __any(!(largest(largest(0.f, qa), qc) < kMostQK));
            const Operand3 q = operand3(split(qa), split(qc));
            const __amdgpu_buffer_rsrc_t rk = make_rsrc((const char*)p.k + tile, tile_bytes);
            // Four key blocks at a time: their additive term is requested in front of their score products, which outlast its
            // way from L2.
            const uint32_t off_b = rb.bf16 ? (2u * (rb.hbase + (uint32_t)(16 * qb + n) * L + 4u * g)) & ~3u : ((uint32_t)(16 * qb + n) * L + 4u * g) * 4u;
            const uint32_t off_m = msk.labels ? 16u * g : ((uint32_t)(16 * qb + n) * L + 4u * g) * 4u, step_b = rb.bf16 ? 32u : 64u;
            const bool odd = ((rb.hbase + (uint32_t)(16 * qb + n) * L + 4u * g) & 1u) != 0;
            const int lq = BM ? load_i32(msk.r, (uint32_t)(16 * qb + n) * 4u) : 0;
            f32x4 tb[2][4], tm[2][4];
            auto request_term = [&](int j0) {
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (j0 + b < NB) {
                        tb[(j0 / 4) & 1][b] = load_f32x4(rb.r, off_b + step_b * (j0 + b));
                        if (BM && has_msk) tm[(j0 / 4) & 1][b] = load_f32x4(msk.r, off_m + 64u * (j0 + b));
                    }
            };
            if (BM) request_term(0);
            auto k_rows = [&](int jb) {
                const char* const row = lk + (16 * jb + n) * 64 + 16 * g;
                return Operand3{*reinterpret_cast<const bf16x8*>(row), *reinterpret_cast<const bf16x8*>(row + SLAB), *reinterpret_cast<const bf16x8*>(row + 2 * SLAB)};
            };
            f32x4 s[NB];
            float m = -INFINITY;
#pragma unroll
            for (int j0 = 0; j0 < NB; j0 += 4) {
                __builtin_amdgcn_sched_barrier(0);
                if (BM && j0 + 4 < NB) request_term(j0 + 4);
                const int j1 = j0 + 4 < NB ? j0 + 4 : NB;
                if (!fp32) {
                    Operand3 k = k_rows(j0);
#pragma unroll
                    for (int jb = j0; jb < j1; ++jb) {
                        const Operand3 c = k;
                        if (jb + 1 < j1) k = k_rows(jb + 1);
                        s[jb] = mfma_bf16(c.h, q.h, small_products(c, q, zero));  // S[16 qb + n][16 jb + 4g + r]
                    }
                } else {
#pragma unroll
                    for (int jb = j0; jb < j1; ++jb) {
                        const uint32_t off = (uint32_t)(16 * jb + n) * here(row_bytes) + 32u * g;  // not kept beside the split path
                        const f32x4 ka = load_f32x4(rk, off), kc = load_f32x4(rk, off + 16u);
                        f32x4 a = zero;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float k0 = ka[i], k1 = kc[i], q0 = qa[i], q1 = qc[i];
                            a = mfma_f32(k1, q1, mfma_f32(k0, q0, a));
                        }
                        s[jb] = a;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                f32x4 (&add)[4] = tb[(j0 / 4) & 1];
                if (BM) {
                    f32x4 (&mk)[4] = tm[(j0 / 4) & 1];
                    if (rb.bf16) {
#pragma unroll
                        for (int b = 0; b < 4; ++b) add[b] = bf16_quad(add[b], odd);
                    }
                    if (has_msk) {
                        if (msk.labels) {
#pragma unroll
                            for (int b = 0; b < 4; ++b) mk[b] = mask_of_labels(lq, __builtin_bit_cast(i32x4, mk[b]), msk.value);
                        }
#pragma unroll
                        for (int b = 0; b < 4; ++b) add[b] += mk[b];
                    }
                }
#pragma unroll
                for (int jb = j0; jb < j1; ++jb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float x = BM ? s[jb][r] * p.scale + add[jb - j0][r] : s[jb][r] * p.scale;
                        if (jb == NB - 1 && 16 * jb + 4 * g + r >= L) x = -INFINITY;
                        s[jb][r] = x;
                        m = fmaxf(m, x);
                    }
            }
            if (qb + (int)parts * W < NB) {  // the wave's next Q rows
                const uint32_t off_q = (uint32_t)(16 * (qb + (int)parts * W) + n) * row_bytes + 32u * g;
                qa = load_f32x4(rq, off_q);
                qc = load_f32x4(rq, off_q + 16u);
            }
            m = max_over_g(m);
            // One fma and exponential per score, with the rounding of mb a factor that the division takes out again -- as long
            // as it is small against 1 (2^-4 at 2^20).  Beyond that the largest score comes off first, which is exact next to it:
            // scores of 1e10, or a row masked out by the type's lowest value, whose mb is infinite.  (Always subtracting:
            // 0.7 % more time over 50 calls.)
            float mb = m * kLog2e;
            if (__any(!(fabsf(m) < 0x1p20f))) {
                subtract_rounded(s, m);
                mb = 0.f;
            }
            float sum = 0.f;
            // Split, the weights are lifted like V (1.4 % of the time; as a multiplication it took registers that spilled)
            auto exponentials = [&](int jb, int lift) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float e = ldexpf(__builtin_amdgcn_exp2f(fmaf(s[jb][r], kLog2e, -mb)), lift);
                    sum += e;
                    s[jb][r] = e;
                }
            };
            f32x4 o0 = zero, o1 = zero;  // O[16 qb + n][4g + r], O[16 qb + n][16 + 4g + r]
            if (!wide) {
                f32x4 t0 = zero, t1 = zero;  // the small terms of both
                const uint16_t* const lv16 = reinterpret_cast<const uint16_t*>(lv) + (4 * g + (n >> 2)) * 32 + 4 * (n & 3);
                constexpr uint32_t P16 = SLAB / 2;
                auto weights = [&](int kp) {  // of a pair of key blocks, in parts
                    const bool two = 2 * kp + 1 < NB;
                    exponentials(2 * kp, kLiftBits);
                    if (two) exponentials(2 * kp + 1, kLiftBits);
                    Planes second = {u32x2{0u, 0u}, u32x2{0u, 0u}, u32x2{0u, 0u}};
                    if (two) second = split(s[two ? 2 * kp + 1 : 0]);
                    return operand3(split(s[2 * kp]), second);
                };
                Operand3 e, next;
                if (MATRIX) e = weights(0);
#pragma unroll
                for (int kp = 0; kp < NB2; ++kp) {
                    const bool two = 2 * kp + 1 < NB;
                    const uint16_t* const v = lv16 + 32 * kp * 32;
                    const bf16x8 h0 = operand_tr(v, 512, two), h1 = operand_tr(v + 16, 512, two);
                    const bf16x8 m0 = operand_tr(v + P16, 512, two), m1 = operand_tr(v + P16 + 16, 512, two);
                    const bf16x8 l0 = operand_tr(v + 2 * P16, 512, two), l1 = operand_tr(v + 2 * P16 + 16, 512, two);
                    if (!MATRIX) e = weights(kp);
                    else if (kp + 1 < NB2) next = weights(kp + 1);
                    // (in the order of small_products, each half on its own: even to 5 % slower, at 12 x 12 with a bias)
                    t0 = mfma_bf16(l0, e.h, t0);
                    t1 = mfma_bf16(l1, e.h, t1);
                    o0 = mfma_bf16(h0, e.h, o0);
                    o1 = mfma_bf16(h1, e.h, o1);
                    t0 = mfma_bf16(m0, e.m, t0);
                    t1 = mfma_bf16(m1, e.m, t1);
                    t0 = mfma_bf16(m0, e.h, t0);
                    t1 = mfma_bf16(m1, e.h, t1);
                    t0 = mfma_bf16(h0, e.m, t0);
                    t1 = mfma_bf16(h1, e.m, t1);
                    t0 = mfma_bf16(h0, e.l, t0);
                    t1 = mfma_bf16(h1, e.l, t1);
                    if (MATRIX && kp + 1 < NB2) e = next;
                    __builtin_amdgcn_sched_barrier(0);
                }
                o0 = (o0 + t0) * (1.0f / kLift);  // the lift of the weights leaves with their sum
                o1 = (o1 + t1) * (1.0f / kLift);
            } else {
                int at = lane;
                asm volatile("" : "+v"(at));  // or the address is kept in a register over the loop
                const float* const v = reinterpret_cast<const float*>(lv + (at >> 4) * (4 * kRowV)) + (at & 15);
                asm volatile("" : "+v"(mb));  // or the exponentials of both paths are taken in front of the branch
#pragma unroll
                for (int jb = 0; jb < NB; ++jb) {
                    exponentials(jb, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float a = v[(16 * jb + r) * (kRowV / 4)], b = v[(16 * jb + r) * (kRowV / 4) + 16], e = s[jb][r];
                        o0 = mfma_f32(a, e, o0);
                        o1 = mfma_f32(b, e, o1);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            sum = sum_over_g(sum);
            const uint32_t off_o = (uint32_t)(16 * qb + n) * row_out + 16u * g;
            const float inv = 1.0f / sum;
            store_f32x4(o0 * inv, ro, off_o);
            store_f32x4(o1 * inv, ro, off_o + 64);
        }
        __syncthreads();  // every wave is done with this tile's slabs
    }
}

template <int NB, bool BM, int W, bool MATRIX = f32_rows_matrix(NB, BM, W)>
hipError_t launch_rows_w(const FwdArgs& a, hipStream_t st) {
    static std::atomic<int> once{0};
    int per_cu = 1;
    const hipError_t e = workgroups_per_cu(reinterpret_cast<const void*>(&fwd_f32_rows_kernel<NB, BM, W, MATRIX>), 64u * W, f32_rows_lds<NB>(), once, per_cu);
    if (e != hipSuccess) return e;
    // While the chip holds several workgroups per tile: the query blocks of a tile over them, each with its own copy of K and V
    // (150 tiles of 196 tokens 15.4 -> 13.9 us), down to one block per SIMD (with two for half of them 8.7 -> 11.1).
    const long long pairs = a.N * a.heads, resident = (long long)cu_count() * per_cu;
    const long long parts = W > f32_rows_waves(NB, BM) ? 1LL : std::max(1LL, std::min(resident / pairs, (long long)(NB + 3) / 4));
    const long long tiles = pairs * parts;
    const unsigned grid = (unsigned)std::min(tiles, resident);
    hipLaunchKernelGGL((fwd_f32_rows_kernel<NB, BM, W, MATRIX>), dim3(grid), dim3(64u * W), f32_rows_lds<NB>(), st, a, (uint32_t)parts, (uint32_t)tiles);
    return hipGetLastError();
}
template <int NB, bool BM>
hipError_t launch_rows_bm(const FwdArgs& a, hipStream_t st) {
    if constexpr (NB == 7) {
        // More tiles than half the CUs but not more than those: a wave per block.  Of two workgroups of four waves per tile some
        // CUs get both, and split K and V twice (200 tiles of 100 tokens, bias 9.0 -> 7.1 us, without 6.7 -> 6.2).  Up to half
        // the CUs each of the two has one to itself; beyond one tile per CU seven waves leave no room for a second workgroup.
        // (At 5, 6 and 8 blocks the two workgroups were no slower than the fp32 instruction; here they were, 7.9 us.)
        const long long pairs = a.N * a.heads;
        if (2 * pairs > cu_count() && pairs <= cu_count()) return launch_rows_w<NB, BM, NB>(a, st);
    }
    if constexpr (!BM && (NB == 6 || NB == 7)) {
        // Up to half a tile per CU a wave has one block and nothing to make beside its products: the remainder's way through the matrix
        // core shows (64 tiles of 112 tokens 4.89 us with it, 4.70 without; 192 tiles 6.07 and 6.17, 1536 tiles 28.0 and 29.3).
        if (2 * a.N * a.heads <= cu_count()) return launch_rows_w<NB, BM, f32_rows_waves(NB, BM), false>(a, st);
    }
    return launch_rows_w<NB, BM, f32_rows_waves(NB, BM)>(a, st);
}
template <int NB>
hipError_t launch_rows(const FwdArgs& a, hipStream_t st) {
    return a.bias || has_mask(a) ? launch_rows_bm<NB, true>(a, st) : launch_rows_bm<NB, false>(a, st);
}

}  // namespace

hipError_t launch_forward_f32_rows(const FwdArgs& a, hipStream_t s) {
    switch ((a.L + 15) / 16) {
        case 5: return launch_rows<5>(a, s);
        case 6: return launch_rows<6>(a, s);
        case 7: return launch_rows<7>(a, s);
        case 8: return launch_rows<8>(a, s);
        case 9: return launch_rows<9>(a, s);
        case 10: return launch_rows<10>(a, s);
        case 11: return launch_rows<11>(a, s);
        case 12: return launch_rows<12>(a, s);
        case 13: return launch_rows<13>(a, s);
        case 14: return launch_rows<14>(a, s);
        case 15: return launch_rows<15>(a, s);
        case 16: return launch_rows<16>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fwa
