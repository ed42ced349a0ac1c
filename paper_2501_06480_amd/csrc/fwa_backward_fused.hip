// Backward (paper Algorithm 2) for 64 < L <= 256 without dBias in one launch, for calls of few tiles.
//
// A workgroup of W = 4 (NB <= 10) or 8 waves (NB = ceil(L / 16) blocks of 16 rows) owns one head, parks the K, V, Q, dO
// slabs of the current window in LDS and walks the windows bw, bw + G, ...  Per window the score tile is produced twice,
// block by block, and never stored:
//
//   pass 1, wave <-> 16-query blocks qb = wave, wave + W, ... ("query on the lane": lane (g, n), slot r of key block
//   jb stands for query 16 qb + n and key 16 jb + 4g + r): scores, softmax statistics M_i and delta_i to LDS, dQ
//   pass 2, wave <-> 16-key blocks jb = wave, wave + W, ... ("key on the lane": lane (g, n), slot r of query block qb
//   stands for query 16 qb + 4g + r and key 16 jb + n): P = exp2(score - M_i), dS = P (dP - delta_i), dV, dK
//
// P and dS enter the matrix cores as hi + lo bf16 pairs (16 significant bits).  What bounds it is the instruction stream of a SIMD, and
// the remainders after the upper parts come from the matrix core: no additive term, 256 windows of 16 x 16 tokens, 4 heads 74.3 -> 71.1 us
// against masks and subtractions, 512 of 12 x 12 62.6 -> 60.0, 864 of 9 x 9, 3 heads 44.9 -> 43.5.
//
// The pair of kernels in fwa_backward_large.hip does the same work in two launches whose waves keep the additive term in
// registers over the windows they walk.  Where a workgroup has a window or two, or there is no term, there is nothing to
// keep, and a second launch and a second fetch of the slabs are what is left of it.  The rule and both sides' times stand
// at fused_pays.
//
// Additive term: in pass 2 a lane needs B[i][j] for 4 queries and one key, 16 lanes cover 16 consecutive keys: dword
// loads, 64 contiguous bytes per 16 lanes.  In pass 1 a lane needs 4 consecutive keys of one query row and neighbouring
// lanes sit in different rows, which the memory pipeline serves a lane at a time; there the wave copies 16 rows x 64
// columns at a time with row-contiguous 16-byte loads into a private LDS patch and picks its values from there.
#include "fwa_device.h"
#include "fwa_internal.h"
#include "fwa_softmax.h"

#include <type_traits>

namespace fwa {
namespace {

struct FusedGeom {
    uint32_t heads, G;
    uint32_t xcd_q, xcd_r;
};

constexpr int fused_waves(int nb) { return nb <= 10 ? 4 : 8; }
// slab rows in 16-byte units: 64 bytes of data and no padding (reads run at the same rate with 16 bytes of it)
constexpr uint32_t kFusedStride = 4;

// HB: no bias (0) or an fp32 bias (1; a bf16 bias arrives as an fp32 copy made once per call); HM: no mask (0), a dense
// mask (1), or region labels from which the mask values are formed in registers (2).  What is absent costs neither
// loads nor registers.
template <int NB, int HB, int HM>
__global__ void __launch_bounds__(64 * fused_waves(NB)) bwd_bf16_fused_kernel(BwdArgs p, FusedGeom gm) {
    constexpr bool BM = HB != 0 || HM != 0;
    constexpr int W = fused_waves(NB);
    constexpr int NB2 = (NB + 1) / 2;
    constexpr int ROWS = 16 * NB;
    constexpr int PASSES = (ROWS + 16 * W - 1) / (16 * W);  // the workgroup moves 16 W slab rows per pass
    constexpr uint32_t STRIDE = kFusedStride;                // slab row in 16-byte units
    constexpr uint32_t SROW = STRIDE * 8;                    // the same in bf16 elements
    constexpr uint32_t SG = 68;                              // patch row: 64 floats + 4 of padding
    extern __shared__ __attribute__((aligned(16))) uint4 lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lb = xcd_logical_block(blockIdx.x, gm.xcd_q, gm.xcd_r);  // heads of a window: one XCD
    const uint32_t h = lb % gm.heads, bw = lb / gm.heads;
    const int L = p.L;
    // token rows are p.ldq (q, k, v), p.ldg (d_o), p.ldd (dq, dk, dv) elements apart; window w starts at row w L
    const uint32_t row_bytes = (uint32_t)p.ldq * 2u, row_g = (uint32_t)p.ldg * 2u, row_d = (uint32_t)p.ldd * 2u;
    const float sl2 = p.scale * kLog2e;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const bf16x4 minus_one = minus_identity(g, n);

    // LDS: slabs [K][V][Q][dO], each [ROWS][STRIDE] uint4; M[ROWS], delta[ROWS]; one patch per wave
    uint4* const lk = lds;
    uint4* const lv = lds + ROWS * STRIDE;
    uint4* const lq = lds + 2 * ROWS * STRIDE;
    uint4* const lg = lds + 3 * ROWS * STRIDE;
    float* const stM = reinterpret_cast<float*>(lds + 4 * ROWS * STRIDE);
    float* const stD = stM + ROWS;
    float* const patch = stD + ROWS + wave * (16 * SG);

    const uint32_t ll = (uint32_t)L * L * 4u;
    const float* const bias32 = static_cast<const float*>(p.bias);
    const __amdgpu_buffer_rsrc_t rb =
        HB == 1 ? make_rsrc(bias32 + (size_t)h * L * L, ll) : make_rsrc(nullptr, 0);

    const uint32_t srow = (uint32_t)tid >> 2, scol = (uint32_t)tid & 3u;  // slab movement: (row, 16 B column)
    const uint32_t tile_bytes = (uint32_t)(L - 1) * row_bytes + 2u * kHeadDim;
    const uint32_t trs = (4u * g + (n >> 2)) * SROW + 4u * (n & 3);  // transposing-read base inside a slab
    const uint32_t opd = (uint32_t)n * STRIDE + g;                   // row operand of block b: slab[opd + 16 b STRIDE]
    const uint32_t tile_bytes_g = (uint32_t)(L - 1) * row_g + 2u * kHeadDim;
    const uint32_t tile_bytes_d = (uint32_t)(L - 1) * row_d + 2u * kHeadDim;
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    // 16 output rows of this wave (64 bytes each: channels 0..15 in `lo`, 16..31 in `hi`, accumulator
    // order) leave through the wave's patch area, free whenever a block's results are ready: written
    // there, read back 16 bytes per lane, one store of 64-byte row pieces instead of two of 32.
    auto store_rows = [&](const u32x2_t lo, const u32x2_t hi, const __amdgpu_buffer_rsrc_t dst, int blk) {
        char* const cell = reinterpret_cast<char*>(patch);
        *reinterpret_cast<u32x2_t*>(cell + n * 80 + g * 8) = lo;
        *reinterpret_cast<u32x2_t*>(cell + n * 80 + 32 + g * 8) = hi;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint32_t r = (uint32_t)(lane >> 2), c = (uint32_t)(lane & 3);
        const u32x4 rows = *reinterpret_cast<const u32x4*>(cell + r * 80 + c * 16);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_raw_buffer_store_b128(rows, dst, (uint32_t)(16 * blk + r) * row_d + 16u * c, 0, 0);
    };
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

    // The slabs of the next window are requested into registers by every wave right before its last stores of the
    // current one -- the big temporaries of the passes are dead by then --, so that their way through memory
    // overlaps with those stores and with the wait for the slowest wave; they are parked between the two barriers
    // that separate the windows.
    u32x4 pk[PASSES], pv[PASSES], pq[PASSES], pg[PASSES];
    auto request = [&](uint32_t w) {
        const size_t tile = ((size_t)w * L * p.ldq + (size_t)h * kHeadDim) * 2u;
        const size_t tile_g = ((size_t)w * L * p.ldg + (size_t)h * kHeadDim) * 2u;
        const __amdgpu_buffer_rsrc_t rk = make_rsrc((const char*)p.k + tile, tile_bytes);
        const __amdgpu_buffer_rsrc_t rv = make_rsrc((const char*)p.v + tile, tile_bytes);
        const __amdgpu_buffer_rsrc_t rq = make_rsrc((const char*)p.q + tile, tile_bytes);
        const __amdgpu_buffer_rsrc_t rg = make_rsrc((const char*)p.d_o + tile_g, tile_bytes_g);
#pragma unroll
        for (int t = 0; t < PASSES; ++t) {
            const uint32_t off = (16 * W * t + srow) * row_bytes + scol * 16u;  // rows beyond L arrive as zeros
            pk[t] = __builtin_amdgcn_raw_buffer_load_b128(rk, off, 0, 0);
            pv[t] = __builtin_amdgcn_raw_buffer_load_b128(rv, off, 0, 0);
            pq[t] = __builtin_amdgcn_raw_buffer_load_b128(rq, off, 0, 0);
            pg[t] = __builtin_amdgcn_raw_buffer_load_b128(rg, (16 * W * t + srow) * row_g + scol * 16u, 0, 0);
        }
    };
    auto park = [&]() {
#pragma unroll
        for (int t = 0; t < PASSES; ++t) {
            const uint32_t row = 16 * W * t + srow;
            if (row < (uint32_t)ROWS) {
                lk[row * STRIDE + scol] = __builtin_bit_cast(uint4, pk[t]);
                lv[row * STRIDE + scol] = __builtin_bit_cast(uint4, pv[t]);
                lq[row * STRIDE + scol] = __builtin_bit_cast(uint4, pq[t]);
                lg[row * STRIDE + scol] = __builtin_bit_cast(uint4, pg[t]);
            }
        }
    };
    if (bw < (uint32_t)p.N) {
        request(bw);
        park();
    }

    for (uint32_t w = bw; w < (uint32_t)p.N; w += gm.G) {
        const size_t tile_d = ((size_t)w * L * p.ldd + (size_t)h * kHeadDim) * 2u;
        const bool has_next = w + gm.G < (uint32_t)p.N;
        __syncthreads();  // the slabs are in place
        // dead until the request at the end of this window: said so, or the compiler carries the old values
        // through both passes on behalf of the path on which no request happens
#pragma unroll
        for (int t = 0; t < PASSES; ++t) pk[t] = pv[t] = pq[t] = pg[t] = u32x4{0u, 0u, 0u, 0u};
        // the labels of the window's tokens when the mask comes as labels
        const __amdgpu_buffer_rsrc_t rl =
            HM == 2 ? make_rsrc(p.labels + (size_t)(w % (uint32_t)p.nW) * L, (uint32_t)L * 4u) : make_rsrc(nullptr, 0);

        // ---------------- pass 1: query blocks wave, wave + W ----------------
        for (int qb = (int)wave; qb < NB; qb += W) {
            const bf16x8 qop = __builtin_bit_cast(bf16x8, lq[opd + 16 * qb * STRIDE]);
            const bf16x8 gop = __builtin_bit_cast(bf16x8, lg[opd + 16 * qb * STRIDE]);
            // rows 16 qb .. 16 qb + 15 of (bias + mask), 64 columns at a time: lane -> (row 4t + lane / 16,
            // columns 4 (lane % 16) ..), 256 contiguous bytes per 16 lanes; rows beyond L lie outside the
            // descriptors and read as zero, columns beyond L are overwritten with -inf below.  The first
            // patch is requested before the products are formed, each further one a patch ahead.
            const uint32_t prow = (uint32_t)lane >> 4, pcol = 4u * ((uint32_t)lane & 15u);
            constexpr int CH = (NB + 3) / 4;
            f32x4 tb[2][4], tm[2][4];
            i32x4 tk[2];  // with labels: those of a patch's 4 columns ...
            int tq[4];    // ... and of the lane's 4 patch rows
            const uint32_t qrow = (uint32_t)(16 * qb) * L * 4u;  // < ll: the block starts inside the tile
            const __amdgpu_buffer_rsrc_t rbq = HB == 1 ? make_rsrc(bias32 + (size_t)h * L * L + (size_t)16 * qb * L, ll - qrow) : rb;
            const __amdgpu_buffer_rsrc_t rmq =
                HM == 1 ? make_rsrc(p.mask + (size_t)(w % (uint32_t)p.nW) * L * L + (size_t)16 * qb * L, ll - qrow) : rb;
            if (HM == 2) {
#pragma unroll
                for (int t = 0; t < 4; ++t) tq[t] = load_i32(rl, (uint32_t)(16 * qb + 4 * t + prow) * 4u);
            }
            auto request_patch = [&](int ch, int slot) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint32_t off = ((uint32_t)(4 * t + prow) * L + pcol) * 4u + 256u * ch;
                    if (HB == 1) tb[slot][t] = load_f32x4(rbq, off);
                    if (HM == 1) tm[slot][t] = load_f32x4(rmq, off);
                }
                if (HM == 2) tk[slot] = load_i32x4(rl, (pcol + 64u * ch) * 4u);
            };
            if (BM) request_patch(0, 0);
            f32x4 s[NB];
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
                s[jb] = mfma_bf16(__builtin_bit_cast(bf16x8, lk[opd + 16 * jb * STRIDE]), qop, zero);
            if (BM) {
#pragma unroll
                for (int ch = 0; ch < CH; ++ch) {
                    const int cur = ch & 1;
                    if (ch + 1 < CH) request_patch(ch + 1, cur ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const f32x4 mk = HM == 2 ? mask_of_labels(tq[t], tk[cur], p.mask_value) : tm[cur][t];
                        const f32x4 bq = tb[cur][t];
                        *reinterpret_cast<f32x4*>(patch + (4 * t + prow) * SG + pcol) =
                            (HB && HM ? bq + mk : (HB ? bq : mk)) * kLog2e;
                    }
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const int jb = 4 * ch + b;
                        if (jb < NB) {
                            const f32x4 a = *reinterpret_cast<const f32x4*>(patch + n * SG + 16 * b + 4 * g);
#pragma unroll
                            for (int r = 0; r < 4; ++r) s[jb][r] = fmaf(s[jb][r], sl2, a[r]);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int jb = 0; jb < NB; ++jb) s[jb] *= sl2;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (16 * (NB - 1) + 4 * g + r >= L) s[NB - 1][r] = -INFINITY;
            float m = s[0][0];
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
                m = fmaxf(fmaxf(m, s[jb][0]), s[jb][1]);
                m = fmaxf(fmaxf(m, s[jb][2]), s[jb][3]);
            }
            m = max_over_g(m);
            float sum = 0.f;
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float e = __builtin_amdgcn_exp2f(s[jb][r] - m);
                    s[jb][r] = e;
                    sum += e;
                }
            sum = sum_over_g(sum);
            const float inv = __builtin_amdgcn_rcpf(sum);
            // s keeps exp(score - max), not normalised: P = s * inv enters delta here and dQ at the very
            // end (one factor per output element instead of one per score)
            float delta = 0.f;
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
                const f32x4 dp = mfma_bf16(__builtin_bit_cast(bf16x8, lv[opd + 16 * jb * STRIDE]), gop, zero);
#pragma unroll
                for (int r = 0; r < 4; ++r) delta = fmaf(s[jb][r], dp[r], delta);
            }
            delta = sum_over_g(delta) * inv;
            if (g == 0) {
                // p_ij = exp2(score_ij - M_i).  With labels a row beyond L gets what makes its probabilities zeros in pass 2,
                // whatever its own scores were: a mask value of -inf may have made them NaN.
                const bool pad = HM == 2 && 16 * qb + n >= L;
                stM[16 * qb + n] = pad ? INFINITY : m + __builtin_amdgcn_logf(sum);
                stD[16 * qb + n] = pad ? 0.f : delta;
            }
            // dQ^T = K^T dS^T over pairs of key blocks; the operands of the next pair are fetched ahead
            f32x4 q0 = zero, q1 = zero;  // dQ[16 qb + n][4g + r], dQ[16 qb + n][16 + 4g + r]
            const uint16_t* lk16 = reinterpret_cast<const uint16_t*>(lk) + trs;
            bf16x8 ov[2][2], tk0[2], tk1[2];
            auto fetch1 = [&](int kp, int slot) {
                const bool two = 2 * kp + 1 < NB;
                ov[slot][0] = __builtin_bit_cast(bf16x8, lv[opd + 16 * (2 * kp) * STRIDE]);
                if (two) ov[slot][1] = __builtin_bit_cast(bf16x8, lv[opd + 16 * (2 * kp + 1) * STRIDE]);
                tk0[slot] = operand_tr(lk16 + (32 * kp) * SROW, 16 * SROW, two);
                tk1[slot] = operand_tr(lk16 + (32 * kp) * SROW + 16, 16 * SROW, two);
            };
            fetch1(0, 0);
#pragma unroll
            for (int kp = 0; kp < NB2; ++kp) {
                const bool two = 2 * kp + 1 < NB;
                const int cur = kp & 1;
                if (kp + 1 < NB2) fetch1(kp + 1, cur ^ 1);
                __builtin_amdgcn_sched_barrier(0);
                bf16x4 hi[2], lo[2];
                hi[1] = lo[1] = as_bf16x4(uint2{0u, 0u});
                f32x4 dp[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (u == 1 && !two) break;
                    dp[u] = mfma_bf16(ov[cur][u], gop, zero);
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (u == 1 && !two) break;
                    const int jb = 2 * kp + u;
                    f32x4 ds;
#pragma unroll
                    for (int r = 0; r < 4; ++r) ds[r] = s[jb][r] * (dp[u][r] - delta);
                    hi[u] = packed4(ds);
                    lo[u] = packed4(remainder(minus_one, hi[u], ds));
                }
                const bf16x8 dh = pair_operand(hi[0], hi[1]), dl = pair_operand(lo[0], lo[1]);
                q0 = mfma_bf16(tk0[cur], dh, q0);
                q1 = mfma_bf16(tk1[cur], dh, q1);
                q0 = mfma_bf16(tk0[cur], dl, q0);
                q1 = mfma_bf16(tk1[cur], dl, q1);
                __builtin_amdgcn_sched_barrier(0);
            }
            const float qs = p.scale * inv;  // the lane's query row: dQ_i = scale / sum_i * (the products above)
            const u32x2 lo2 = {pack_bf16(q0[0] * qs, q0[1] * qs), pack_bf16(q0[2] * qs, q0[3] * qs)};
            const u32x2 hi2 = {pack_bf16(q1[0] * qs, q1[1] * qs), pack_bf16(q1[2] * qs, q1[3] * qs)};
            store_rows(lo2, hi2, make_rsrc((char*)p.dq + tile_d, tile_bytes_d), qb);
        }
        __syncthreads();

        // ---------------- pass 2: key blocks wave, wave + W, ..., two at a time ----------------
        // A wave that owns two key blocks works on both at once: every operand it fetches for a query
        // block (Q and dO rows, their transposes, the statistics) then serves two key blocks, which
        // halves the LDS traffic of this pass, and the two blocks are independent chains of work.
        auto pass2 = [&](auto nk_tag, const int jb0) {
            constexpr int NK = decltype(nk_tag)::value;  // key blocks jb0 (and jb0 + W)
            bf16x8 kop[NK], vop[NK];
            f32x4 v0[NK], v1[NK], k0[NK], k1[NK];  // dV, dK [16 jb + n][4g + r] and [..][16 + 4g + r]
            int lkey[NK];
#pragma unroll
            for (int t = 0; t < NK; ++t) {
                const int jb = jb0 + t * W;
                kop[t] = __builtin_bit_cast(bf16x8, lk[opd + 16 * jb * STRIDE]);
                vop[t] = __builtin_bit_cast(bf16x8, lv[opd + 16 * jb * STRIDE]);
                v0[t] = v1[t] = k0[t] = k1[t] = zero;
                lkey[t] = HM == 2 ? load_i32(rl, (uint32_t)(16 * jb + n) * 4u) : 0;
            }
            // A key beyond L (a lane of the last key block) is not masked out: what it computes -- from
            // zero rows of K and V, possibly an overflow -- stays in its own column of every product,
            // i.e. in rows of dV and dK beyond L, which the stores drop.
            const uint16_t* lg16 = reinterpret_cast<const uint16_t*>(lg) + trs;
            const uint16_t* lq16 = reinterpret_cast<const uint16_t*>(lq) + trs;
            uint32_t aoff[4];  // additive term of query 4g + r and key 16 jb0 + n; key block t: + 64 W t bytes
#pragma unroll
            for (int r = 0; r < 4; ++r) aoff[r] = ((uint32_t)(4 * g + r) * L + 16u * jb0 + n) * 4u;
            // Row operands, statistics (LDS) and additive terms (L2) are fetched one query block ahead of
            // their use, the transposed operands one pair of query blocks ahead; the scheduling barriers
            // keep the compiler from hoisting more than that.
            bf16x8 oq[2], og[2], tg0[2], tg1[2], tx0[2], tx1[2];
            f32x4 oM[2], oD[2], ab[2][NK], am[2][NK];
            i32x4 al[2];
            auto fetch_q = [&](int qb, int slot) {
                oq[slot] = __builtin_bit_cast(bf16x8, lq[opd + 16 * qb * STRIDE]);
                og[slot] = __builtin_bit_cast(bf16x8, lg[opd + 16 * qb * STRIDE]);
                oM[slot] = *reinterpret_cast<const f32x4*>(stM + 16 * qb + 4 * g);
                oD[slot] = *reinterpret_cast<const f32x4*>(stD + 16 * qb + 4 * g);
                if (BM) {
                    // rows beyond L lie outside the descriptors (which start at the first row of the query
                    // block, so that the 4 lane offsets serve every block)
                    const uint32_t qrow = (uint32_t)(16 * qb) * L;
                    const __amdgpu_buffer_rsrc_t rbq = HB == 1 ? make_rsrc(bias32 + (size_t)h * L * L + qrow, ll - 4u * qrow) : rb;
                    const __amdgpu_buffer_rsrc_t rmq =
                        HM == 1 ? make_rsrc(p.mask + (size_t)(w % (uint32_t)p.nW) * L * L + qrow, ll - 4u * qrow) : rb;
#pragma unroll
                    for (int t = 0; t < NK; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            if (HB == 1) ab[slot][t][r] = load_f32(rbq, aoff[r] + 64u * W * t);
                            if (HM == 1) am[slot][t][r] = load_f32(rmq, aoff[r] + 64u * W * t);
                        }
                    // with labels: those of the 4 query rows, compared with the key's where the term is used
                    if (HM == 2) al[slot] = load_i32x4(rl, (uint32_t)(16 * qb + 4 * g) * 4u);
                }
            };
            auto fetch_t = [&](int qp, int slot) {  // dO^T and Q^T of the 32 queries (channel on the lane)
                const bool two = 2 * qp + 1 < NB;
                tg0[slot] = operand_tr(lg16 + (32 * qp) * SROW, 16 * SROW, two);
                tg1[slot] = operand_tr(lg16 + (32 * qp) * SROW + 16, 16 * SROW, two);
                tx0[slot] = operand_tr(lq16 + (32 * qp) * SROW, 16 * SROW, two);
                tx1[slot] = operand_tr(lq16 + (32 * qp) * SROW + 16, 16 * SROW, two);
            };
            fetch_q(0, 0);
            fetch_t(0, 0);
#pragma unroll
            for (int qp = 0; qp < NB2; ++qp) {
                const bool two = 2 * qp + 1 < NB;
                const int tcur = qp & 1;
                if (qp + 1 < NB2) fetch_t(qp + 1, tcur ^ 1);
                bf16x4 ph[NK][2], pl[NK][2], sh[NK][2], sl[NK][2];
#pragma unroll
                for (int t = 0; t < NK; ++t) ph[t][1] = pl[t][1] = sh[t][1] = sl[t][1] = as_bf16x4(uint2{0u, 0u});
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (u == 1 && !two) break;
                    const int qb = 2 * qp + u, cur = qb & 1;
                    if (qb + 1 < NB) fetch_q(qb + 1, cur ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
                    f32x4 sc[NK], dp[NK];
#pragma unroll
                    for (int t = 0; t < NK; ++t) {
                        sc[t] = mfma_bf16(oq[cur], kop[t], zero);  // sc[r] = <q_i, k_j>, i = 16 qb + 4g + r, j = 16 jb + n
                        dp[t] = mfma_bf16(og[cur], vop[t], zero);
                    }
#pragma unroll
                    for (int t = 0; t < NK; ++t) {
                        f32x4 pr, ds;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            float x;
                            if (BM) {
                                const float mk = HM == 2 ? (al[cur][r] == lkey[t] ? 0.f : p.mask_value) : am[cur][t][r];
                                const float bv = ab[cur][t][r];
                                const float add = HB && HM ? bv + mk : (HB ? bv : mk);
                                x = fmaf(sc[t][r], sl2, fmaf(add, kLog2e, -oM[cur][r]));
                            } else {
                                x = fmaf(sc[t][r], sl2, -oM[cur][r]);
                            }
                            pr[r] = __builtin_amdgcn_exp2f(x);
                            ds[r] = pr[r] * (dp[t][r] - oD[cur][r]);
                        }
                        ph[t][u] = packed4(pr);
                        pl[t][u] = packed4(remainder(minus_one, ph[t][u], pr));
                        sh[t][u] = packed4(ds);
                        sl[t][u] = packed4(remainder(minus_one, sh[t][u], ds));
                    }
                }
#pragma unroll
                for (int t = 0; t < NK; ++t) {
                    const bf16x8 PH = pair_operand(ph[t][0], ph[t][1]), PL = pair_operand(pl[t][0], pl[t][1]);
                    const bf16x8 SH = pair_operand(sh[t][0], sh[t][1]), SL = pair_operand(sl[t][0], sl[t][1]);
                    v0[t] = mfma_bf16(tg0[tcur], PH, v0[t]);
                    v1[t] = mfma_bf16(tg1[tcur], PH, v1[t]);
                    k0[t] = mfma_bf16(tx0[tcur], SH, k0[t]);
                    k1[t] = mfma_bf16(tx1[tcur], SH, k1[t]);
                    v0[t] = mfma_bf16(tg0[tcur], PL, v0[t]);
                    v1[t] = mfma_bf16(tg1[tcur], PL, v1[t]);
                    k0[t] = mfma_bf16(tx0[tcur], SL, k0[t]);
                    k1[t] = mfma_bf16(tx1[tcur], SL, k1[t]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // The wave's last key blocks of this window (with 8 waves it comes through here once per window;
            // with 4, up to twice, and asks after the loop below instead).
            if (W == 8 && has_next) request(w + gm.G);
#pragma unroll
            for (int t = 0; t < NK; ++t) {
                const int jb = jb0 + t * W;
                const u32x2 va = {pack_bf16(v0[t][0], v0[t][1]), pack_bf16(v0[t][2], v0[t][3])};
                const u32x2 vb = {pack_bf16(v1[t][0], v1[t][1]), pack_bf16(v1[t][2], v1[t][3])};
                const u32x2 ka = {pack_bf16(k0[t][0] * p.scale, k0[t][1] * p.scale), pack_bf16(k0[t][2] * p.scale, k0[t][3] * p.scale)};
                const u32x2 kb = {pack_bf16(k1[t][0] * p.scale, k1[t][1] * p.scale), pack_bf16(k1[t][2] * p.scale, k1[t][3] * p.scale)};
                store_rows(va, vb, make_rsrc((char*)p.dv + tile_d, tile_bytes_d), jb);
                store_rows(ka, kb, make_rsrc((char*)p.dk + tile_d, tile_bytes_d), jb);
            }
        };
        for (int jb0 = (int)wave; jb0 < NB; jb0 += 2 * W) {
            if (jb0 + W < NB)
                pass2(std::integral_constant<int, 2>{}, jb0);
            else
                pass2(std::integral_constant<int, 1>{}, jb0);
        }
        if (W == 4 && has_next) request(w + gm.G);
        __syncthreads();  // every wave has left the slabs
        if (has_next) park();
    }
}

// Whether this kernel is the faster one for `tiles` tiles of which the device holds `resident` at a time; times in us,
// the pair of kernels against this one, 256 CUs, with bias unless said otherwise:
//   no additive term: always                   L = 144: 35.0 : 31.4 (1024 tiles), 63.2 : 61.9 (2048); L = 256: 157 : 147 (2048)
//   NB <= 8 (two 16-row blocks per wave)       up to three full rounds of resident tiles (NB = 7, 8: four).  L = 81: 14.8 : 11.4
//                                              (512), 28.6 : 27.5 (1536), 34.1 : 35.2 (2048); L = 100: 20.4 : 13.8 (512),
//                                              44.2 : 42.8 (2048), 60.3 : 67.7 (3072)
//   NB = 11                                    up to four rounds.  L = 169: 21.8 : 15.4 (256), 49.8 : 49.0 (1024), 67.7 : 69.8 (1536)
//   the others (9, 10: three blocks for one wave; from 12 on the second block of most waves): only in the first two
//                                              rounds, and where the pair's keys kernel walks two windows in the first, four
//                                              (NB = 9, 10: six) in the second: both sides go up in steps.  (tiles; windows)
//                                              L = 144: 12.7 : 14.3 (64; 1), 24.5 : 21.6 (512; 4), 32.1 : 36.4 (768; 5),
//                                              39.0 : 37.1 (1024; 7); with 16 heads and labels 44.5 : 42.2 (864; 6);
//                                              L = 225, 3 heads 31.4 : 24.2 (144; 2), 8 heads and labels 53.9 : 48.4 (432; 4);
//                                              L = 256: 18.6 : 22.6 (64; 1), 30.8 : 24.7 (256; 2), 39.2 : 44.2 (384; 3),
//                                              48.6 : 44.7 (512; 4), 82.2 : 85.7 (1024)
bool fused_pays(int nb, bool term, long long tiles, long long resident, long long windows) {
    if (!term) return true;
    if (nb <= 6) return tiles <= 3 * resident;
    if (nb <= 8) return tiles <= 4 * resident;
    if (nb == 11) return tiles <= 4 * resident;
    const long long before = (tiles - 1) / resident * resident;  // tiles of the full rounds
    if (before > resident) return false;
    return before > 0 ? windows >= (nb <= 10 ? 6 : 4) : windows >= 2;
}

template <int NB, int HB, int HM>
hipError_t launch_fused_one(const BwdArgs& a, hipStream_t st, bool forced, long long windows, bool& taken) {
    constexpr int W = fused_waves(NB);
    const void* fn = reinterpret_cast<const void*>(&bwd_bf16_fused_kernel<NB, HB, HM>);
    const unsigned block = 64u * W;
    const size_t lds = (size_t)4 * 16 * NB * kFusedStride * 16 + (size_t)2 * 16 * NB * 4 + (size_t)W * 16 * 68 * 4;  // slabs, statistics, one patch per wave
    static std::atomic<int> once{0};
    int per_cu = 1;
    const hipError_t e = workgroups_per_cu(fn, block, lds, once, per_cu);
    if (e != hipSuccess) return e;
    const long long resident = (long long)cu_count() * per_cu;
    taken = forced || fused_pays(NB, HB != 0 || HM != 0, a.N * (long long)a.heads, resident, windows);
    if (!taken) return hipSuccess;
    FusedGeom gm;
    gm.heads = (uint32_t)a.heads;
    long long G = resident / a.heads;  // one resident workgroup per slot and head
    if (G < 1) G = 1;
    if (G > a.N) G = a.N;
    gm.G = (uint32_t)G;
    const unsigned grid = gm.G * gm.heads;
    gm.xcd_q = grid / 8u;
    gm.xcd_r = grid % 8u;
    hipLaunchKernelGGL((bwd_bf16_fused_kernel<NB, HB, HM>), dim3(grid), dim3(block), lds, st, a, gm);
    return hipGetLastError();
}

template <int NB>
hipError_t launch_fused_nb(const BwdArgs& a, hipStream_t st, bool forced, long long windows, bool& taken) {
    if (a.bias) {
        if (a.labels) return launch_fused_one<NB, 1, 2>(a, st, forced, windows, taken);
        return a.mask ? launch_fused_one<NB, 1, 1>(a, st, forced, windows, taken) : launch_fused_one<NB, 1, 0>(a, st, forced, windows, taken);
    }
    if (a.labels) return launch_fused_one<NB, 0, 2>(a, st, forced, windows, taken);
    return a.mask ? launch_fused_one<NB, 0, 1>(a, st, forced, windows, taken) : launch_fused_one<NB, 0, 0>(a, st, forced, windows, taken);
}

}  // namespace

// `taken` tells whether the call was launched: always with `forced`, else where this kernel is the faster one; `windows`: per
// workgroup of the keys kernel, were the pair to run
hipError_t launch_backward_bf16_fused(const BwdArgs& a, hipStream_t st, bool forced, long long windows, bool& taken) {
    taken = false;
    if (a.dbias) return hipSuccess;  // the keys kernel sums it up
    if (a.bias && a.bias_bf16) return hipErrorInvalidValue;  // the caller hands over an fp32 copy
    switch ((a.L + 15) / 16) {
        case 5: return launch_fused_nb<5>(a, st, forced, windows, taken);
        case 6: return launch_fused_nb<6>(a, st, forced, windows, taken);
        case 7: return launch_fused_nb<7>(a, st, forced, windows, taken);
        case 8: return launch_fused_nb<8>(a, st, forced, windows, taken);
        case 9: return launch_fused_nb<9>(a, st, forced, windows, taken);
        case 10: return launch_fused_nb<10>(a, st, forced, windows, taken);
        case 11: return launch_fused_nb<11>(a, st, forced, windows, taken);
        case 12: return launch_fused_nb<12>(a, st, forced, windows, taken);
        case 13: return launch_fused_nb<13>(a, st, forced, windows, taken);
        case 14: return launch_fused_nb<14>(a, st, forced, windows, taken);
        case 15: return launch_fused_nb<15>(a, st, forced, windows, taken);
        case 16: return launch_fused_nb<16>(a, st, forced, windows, taken);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fwa
