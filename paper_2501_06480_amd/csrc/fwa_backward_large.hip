// Backward (paper Algorithm 2) for 64 < L <= 256: the score matrix of a tile no longer fits
// the registers of a few waves, so it is produced twice, block by block, in the two
// orientations the two kinds of output need, by two kernels, and never leaves the registers.
//
//   rows kernel, wave <-> one block of 16 queries ("query on the lane": lane (g, n), slot r of key block jb stands for
//   query 16 qb + n and key 16 jb + 4g + r):
//       S^T = K Q^T for all key blocks, + bias + mask, row max, exp, row sum
//       delta_i = sum_j P_ij dP_ij with dP^T = V dO^T produced block by block
//       dQ rows of the block: dS^T is already the operand of dQ^T = K^T dS^T (dP recomputed
//       block by block; K^T through the transposing LDS read)
//       M_i = max_i + log2(sum_i) and -delta_i of the block's rows for the other kernel
//   keys kernel, wave <-> one block of 16 keys ("key on the lane": lane (g, n), slot r of query block qb
//   stands for query 16 qb + 4g + r and key 16 jb + n):
//       S = Q K^T and dP = dO V^T block by block, P = exp2(score - M_i), dS = P (dP - delta_i):
//       the accumulator layout is exactly the operand layout of dV^T = dO^T P and dK^T = Q^T dS
//       with the queries on the k-slots, so P and dS go straight back into the matrix cores;
//       with DB, dS is added to dBias[all queries][the wave's keys], held in registers across windows.
//
// Nothing is transposed and no L x L tile is ever stored; the price is a second S / dP / exp.
// Calls without dBias in which there is little to keep from window to window run in one launch (fwa_backward_fused.hip).
// P and dS enter the matrix cores as hi + lo bf16 pairs (16 significant bits), as in the
// kernels for small windows.
//
// Both kernels are persistent: a wave keeps its block for life and its workgroup walks the windows bw, bw + G, ...
// Most of their work is vector instructions (6 to 7 per score besides the exponential), so everything that does not
// change from window to window stays out of the loop:
// (bias + mask[w mod nW]) * log2e of the block's 16 x L scores sits in registers (G is a multiple of the mask
// period), -delta_i enters as the accumulator that the product dO V^T starts from.  (-M_i / scale as that of Q K^T saves a subtraction
// per score, 0 to 4 % of a call, but rounds every score at the size of M: the probability of a key that holds its row
// alone was off by 1 % at scores of 1e5 and by any factor beyond 1e6.)  Reading the additive term per window
// instead (the form for dense masks whose period no G is a multiple of) costs its loads, the LDS patch that turns
// rows into lanes, and three to four more instructions per score.  Measured, N = 1024 windows of 16 x 16 tokens,
// 4 heads, bias + labels + dBias: rows 210 -> 148 us, keys 283 -> 167 us (kernels of their own that read the term per
// window and parked the slabs out of registers between two barriers), the whole call 465 -> 325 us; N = 315 windows
// of 14 x 14, 5 heads, bias, no dBias: 133 (one kernel with both passes) -> 51 + 55 us.  What bounds them is the instruction
// stream of a SIMD: a matrix instruction takes 8 to 11 cycles from the vector instructions beside it, and some vector instructions
// (the two-term dot product, which made the remainder of the hi/lo split before) wait for the matrix core to be idle.  With the
// remainder from the matrix core the call takes 298 us instead of 314, 14 x 14 windows without dBias 89 instead of 94; the clock falls from
// 1.9 to 1.83 GHz of 2.4 meanwhile (power).  (Exponentials of the scores without their maximum save another 2 to 3 %, but rows whose sum
// they lose have to be made twice: 28 to 38 % of the call at scores of standard deviation 10.)
//
// The statistics M_i, -delta_i (8 bytes per query) travel from one kernel to the other inside the outputs that the
// second one overwrites: the 16 floats of a query block are as long as the 64-byte slice of the head in one token
// row, and every workgroup of the keys kernel finds the statistics of all query blocks in the rows of its own first
// key block -- M in dV, -delta in dK, query block qb in row 16 part + qb -- which it alone reads, and overwrites
// when it has.  So neither kernel needs scratch memory but for the dBias partial sums.
#include "fwa_device.h"
#include "fwa_internal.h"
#include "fwa_softmax.h"

namespace fwa {
namespace {

struct LargeGeom {
    uint32_t heads, parts, G;
    uint32_t xcd_q, xcd_r;
};

// Slab rows in 16-byte units: 64 bytes of data and no padding.  Row-operand and transposing
// reads run at the same rate as with 16 bytes of padding (measured).
constexpr uint32_t kLargeStride = 4;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// The key blocks of a head are spread over the workgroups ("parts") of the keys kernel in turns: wave v of part
// `part` owns key block part + parts * v.  The first block of a part is then always one of the first four, i.e. a
// full one, whose 16 rows have room for the statistics of 16 query blocks.
constexpr int keys_parts(int nb) { return (nb + 3) / 4; }
constexpr int keys_waves(int nb) { return (nb + keys_parts(nb) - 1) / keys_parts(nb); }

// M and -delta of query block qb (lane (g, n) holds those of query 16 qb + n, the same for all g) to every part of
// the keys kernel: lane row g serves part g.
template <int NB>
__device__ __forceinline__ void store_stats(const BwdArgs& p, size_t tile_d, uint32_t row_d, int qb, int n, int g, float M,
                                            float neg_delta) {
    constexpr uint32_t PARTS = (uint32_t)keys_parts(NB);
    // rows 16 part + qb of the head's slice, all below 16 PARTS <= L
    const uint32_t bytes = (16u * PARTS - 1u) * row_d + 64u;
    const uint32_t off = (uint32_t)g < PARTS ? (uint32_t)(16 * g + qb) * row_d + 4u * (uint32_t)n : 0xfffffff0u;
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, M), make_rsrc((char*)p.dv + tile_d, bytes), off, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, neg_delta), make_rsrc((char*)p.dk + tile_d, bytes), off, 0, 0);
}

// 16 output rows of a wave (64 bytes each: channels 0..15 in `lo`, 16..31 in `hi`, accumulator order) leave through
// 16 x 80 bytes of LDS of the wave's own: written there, read back 16 bytes per lane, one store of 64-byte row
// pieces instead of two of 32.
__device__ __forceinline__ void store_rows(char* cell, const u32x2 lo, const u32x2 hi, const __amdgpu_buffer_rsrc_t dst,
                                           int blk, uint32_t row_d, int lane) {
    const int n = lane & 15, g = lane >> 4;
    *reinterpret_cast<u32x2*>(cell + n * 80 + g * 8) = lo;
    *reinterpret_cast<u32x2*>(cell + n * 80 + 32 + g * 8) = hi;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint32_t r = (uint32_t)(lane >> 2), c = (uint32_t)(lane & 3);
    const u32x4 rows = *reinterpret_cast<const u32x4*>(cell + r * 80 + c * 16);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_raw_buffer_store_b128(rows, dst, (uint32_t)(16 * blk + r) * row_d + 16u * c, 0, 0);
}

// What follows the scores in the query orientation, shared by the two rows kernels: s holds the scaled scores (with
// the additive term, -inf beyond L), m their maximum over the lane's keys; on return the block's dQ rows are packed in
// lo2, hi2, and M, neg_delta are its statistics.  lk, lv: the K and V slabs; opd / trs: the lane's offsets for row
// operands / transposing reads.  Matrix products are issued one step ahead of the vector work that needs them, and
// the scheduling barriers keep the compiler from collecting them at one end of a loop (2-3 % at L = 196).
// `between(i)` is called in between, i = 0, 1, ..., NB - 1 (a place for the next window's loads).
// What remains of dS after its upper parts comes from the matrix core and is packed a step later; TIGHT: both parts in one step, the
// remainder by the dot product, in fewer registers.
template <int NB, bool TIGHT, class Between>
__device__ __forceinline__ void rows_block(f32x4 (&s)[NB], float m, const bf16x8 gop, const uint4* lk, const uint4* lv,
                                           uint32_t opd, uint32_t trs, [[maybe_unused]] const bf16x4 minus_one, float scale, float& M,
                                           float& neg_delta, u32x2& lo2, u32x2& hi2, Between between) {
    constexpr int NB2 = (NB + 1) / 2;
    constexpr uint32_t STRIDE = kLargeStride, SROW = STRIDE * 8;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    auto v_rows = [&](int jb) { return __builtin_bit_cast(bf16x8, lv[opd + 16 * jb * STRIDE]); };
    m = max_over_g(m);
    // s keeps exp(score - max), not normalised: P = s / sum enters delta here and dQ at the very
    // end (one factor per output element instead of one per score)
    float sum = 0.f, delta = 0.f;
    f32x4 dp[2];
    dp[0] = mfma_bf16(v_rows(0), gop, zero);
    bf16x8 ov = v_rows(1);
#pragma unroll
    for (int jb = 0; jb < NB; ++jb) {
        __builtin_amdgcn_sched_barrier(0);
        between(jb);
        if (jb + 1 < NB) dp[(jb + 1) & 1] = mfma_bf16(ov, gop, zero);
        if (jb + 2 < NB) ov = v_rows(jb + 2);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float e = __builtin_amdgcn_exp2f(s[jb][r] - m);
            s[jb][r] = e;
            sum += e;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) delta = fmaf(s[jb][r], dp[jb & 1][r], delta);
    }
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 o0 = v_rows(0), o1 = v_rows(1);
    sum = sum_over_g(sum);
    const float inv = __builtin_amdgcn_rcpf(sum);
    delta = sum_over_g(delta) * inv;
    M = m + __builtin_amdgcn_logf(sum);  // p_ij = exp2(score_ij - M_i)
    neg_delta = -delta;
    const f32x4 nd = {neg_delta, neg_delta, neg_delta, neg_delta};
    // dQ^T = K^T dS^T over pairs of key blocks; dP is made anew, from -delta
    f32x4 q0 = zero, q1 = zero;  // dQ[16 qb + n][4g + r], dQ[16 qb + n][16 + 4g + r]
    const uint16_t* lk16 = reinterpret_cast<const uint16_t*>(lk) + trs;
    f32x4 da[2], db[2];  // dP - delta of the two blocks of a pair (TIGHT: of two pairs in turns)
    da[0] = mfma_bf16(o0, gop, nd);
    db[0] = mfma_bf16(o1, gop, nd);
    if (NB > 2) o0 = v_rows(2);
    if (NB > 3) o1 = v_rows(3);
    bf16x8 tk0, tk1;
    u32x4 dh = {0u, 0u, 0u, 0u}, dl = dh;
    [[maybe_unused]] f32x4 ra = zero, rb = zero;  // what remains of dS of the last pair
    auto accumulate = [&]() {
        q0 = mfma_bf16(tk0, as_bf16x8(dh), q0);
        q1 = mfma_bf16(tk1, as_bf16x8(dh), q1);
        if constexpr (!TIGHT)
            dl = u32x4{pack_bf16(ra[0], ra[1]), pack_bf16(ra[2], ra[3]), pack_bf16(rb[0], rb[1]), pack_bf16(rb[2], rb[3])};
        q0 = mfma_bf16(tk0, as_bf16x8(dl), q0);
        q1 = mfma_bf16(tk1, as_bf16x8(dl), q1);
    };
#pragma unroll
    for (int kp = 0; kp < NB2; ++kp) {
        const bool two = 2 * kp + 1 < NB;
        const int cur = TIGHT ? kp & 1 : 0, nxt = TIGHT ? cur ^ 1 : 0;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (TIGHT) {
            if (2 * kp + 2 < NB) da[nxt] = mfma_bf16(o0, gop, nd);
            if (2 * kp + 3 < NB) db[nxt] = mfma_bf16(o1, gop, nd);
            if (kp > 0) accumulate();
            if (2 * kp + 4 < NB) o0 = v_rows(2 * kp + 4);
            if (2 * kp + 5 < NB) o1 = v_rows(2 * kp + 5);
        } else if (kp > 0) {
            accumulate();
        }
        tk0 = operand_tr(lk16 + (32 * kp) * SROW, 16 * SROW, two);
        tk1 = operand_tr(lk16 + (32 * kp) * SROW + 16, 16 * SROW, two);
        const f32x4 a = s[2 * kp] * da[cur], b = two ? s[two ? 2 * kp + 1 : 0] * db[cur] : zero;  // dS, times the row sum
        if constexpr (TIGHT) {
            bf16x4 hi[2], lo[2];
            hi[1] = lo[1] = as_bf16x4(uint2{0u, 0u});
            split_hi_lo_dot(a, hi[0], lo[0]);
            if (two) split_hi_lo_dot(b, hi[1], lo[1]);
            dh = __builtin_bit_cast(u32x4, pair_operand(hi[0], hi[1])), dl = __builtin_bit_cast(u32x4, pair_operand(lo[0], lo[1]));
        } else {
            if (2 * kp + 2 < NB) da[nxt] = mfma_bf16(o0, gop, nd);
            if (2 * kp + 3 < NB) db[nxt] = mfma_bf16(o1, gop, nd);
            if (2 * kp + 4 < NB) o0 = v_rows(2 * kp + 4);
            if (2 * kp + 5 < NB) o1 = v_rows(2 * kp + 5);
            dh = u32x4{pack_bf16(a[0], a[1]), pack_bf16(a[2], a[3]), two ? pack_bf16(b[0], b[1]) : 0u, two ? pack_bf16(b[2], b[3]) : 0u};
            ra = remainder(minus_one, uint2{dh.x, dh.y}, a);
            rb = two ? remainder(minus_one, uint2{dh.z, dh.w}, b) : zero;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    accumulate();
    const float qs = scale * inv;  // the lane's query row: dQ_i = scale / sum_i * (the products above)
    lo2 = u32x2{pack_bf16(q0[0] * qs, q0[1] * qs), pack_bf16(q0[2] * qs, q0[3] * qs)};
    hi2 = u32x2{pack_bf16(q1[0] * qs, q1[1] * qs), pack_bf16(q1[2] * qs, q1[3] * qs)};
}
// -inf for the keys of the last block beyond L; the running maximum m takes a block's scores in
template <int NB>
__device__ __forceinline__ void pad_and_max(f32x4& x, int jb, int L, int g, float& m) {
    if (jb == NB - 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (16 * (NB - 1) + 4 * g + r >= L) x[r] = -INFINITY;
    }
    m = fmaxf(fmaxf(m, x[0]), x[1]);
    m = fmaxf(fmaxf(m, x[2]), x[3]);
}

// ------------------------------------------------------------------ rows kernel
// W waves = W consecutive query blocks of the head (the head is split over two workgroups when NB > 12), K and V of
// the head in a double-buffered LDS slab, the wave's own Q and dO rows straight from global memory as operands.  One
// barrier per window.
// BM: there is an additive term.  PW: the mask comes as labels whose period does not divide G; the bias alone stays
// in registers, the labels of a window travel with its slabs and the mask is formed per score.
constexpr int rows_parts(int nb) { return nb <= 12 ? 1 : 2; }
constexpr int rows_waves(int nb) { return (nb + rows_parts(nb) - 1) / rows_parts(nb); }

template <int NB>
constexpr size_t rows_lds() {
    return (size_t)2 * 2 * 16 * NB * kLargeStride * 16 + (size_t)2 * 16 * NB * 4 + (size_t)rows_waves(NB) * 16 * 80;
}

// Waves per SIMD, said where the compiler would take two registers too many and lose one (112 tokens, bias, 690 windows, 3 heads:
// 42.7 us with four, 45.3 with three; elsewhere its own choice is as fast, and without a term at 81 to 96 and 193 to 224 tokens 3 to 7 %
// faster than one wave more).
constexpr int rows_per_simd(int nb, bool bm, bool pw) { return nb == 7 && bm && !pw ? 4 : 1; }

// Kernels whose three waves per SIMD leave no registers for the longer pipeline (16 to 19 of them spilled): 192 tokens, labels per window,
// 232 windows, 3 heads 44.4 us against 56.4, with dBias 52.9 against 64.4, 161 tokens with dBias 54.9 against 65.8.
constexpr bool rows_tight(int nb, bool pw) { return pw && (nb == 11 || nb == 12); }

template <int NB, bool BM, bool PW>
__global__ void __launch_bounds__(64 * rows_waves(NB), rows_per_simd(NB, BM, PW)) bwd_bf16_rows_kernel(BwdArgs p, LargeGeom gm) {
    constexpr int W = rows_waves(NB);
    constexpr int ROWS = 16 * NB;
    constexpr int PASSES = (ROWS + 16 * W - 1) / (16 * W);  // the workgroup moves 16 W slab rows per pass
    constexpr uint32_t STRIDE = kLargeStride, SROW = STRIDE * 8;
    constexpr uint32_t SLAB = ROWS * STRIDE;                // in uint4
    extern __shared__ __attribute__((aligned(16))) uint4 lds[];  // [2 buffers][K, V][ROWS][STRIDE], labels [2][ROWS], output cells
    const int tid = threadIdx.x, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int* const llab = reinterpret_cast<int*>(lds + 4 * SLAB);
    char* const cell = reinterpret_cast<char*>(llab + 2 * ROWS) + wave * (16 * 80);
    // workgroups that share 128-byte lines (the parts of a head, the heads of a window) are neighbours: one XCD
    const uint32_t lb = xcd_logical_block(blockIdx.x, gm.xcd_q, gm.xcd_r);
    const uint32_t part = lb % gm.parts, bh = lb / gm.parts;
    const uint32_t h = bh % gm.heads, bw = bh / gm.heads;
    const int qb = (int)(part * W + wave);
    const bool active = qb < NB;
    const int L = p.L;
    const uint32_t row_bytes = (uint32_t)p.ldq * 2u, row_g = (uint32_t)p.ldg * 2u, row_d = (uint32_t)p.ldd * 2u;
    const float sl2 = p.scale * kLog2e;
    const bf16x4 minus_one = minus_identity(g, n);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};

    const uint32_t tile_bytes = (uint32_t)(L - 1) * row_bytes + 2u * kHeadDim;
    const uint32_t tile_bytes_g = (uint32_t)(L - 1) * row_g + 2u * kHeadDim;
    const uint32_t tile_bytes_d = (uint32_t)(L - 1) * row_d + 2u * kHeadDim;
    const uint32_t off_q = (uint32_t)(16 * qb + n) * row_bytes + 16u * g;
    const uint32_t off_g = (uint32_t)(16 * qb + n) * row_g + 16u * g;
    const uint32_t trs = (4u * g + (n >> 2)) * SROW + 4u * (n & 3);
    const uint32_t opd = (uint32_t)n * STRIDE + g;

    // K and V go straight from memory into LDS, into the buffer that the current window does not use; the wave's own
    // Q and dO rows (and PW: the labels, 4 tid .. 4 tid + 3) wait in registers.  Rows beyond L are never loaded:
    // zeros from the start.
    static_assert(4 * SLAB * 16 <= 65536, "direct loads reach the first 64 KB");
    const uint32_t off_slab = ((uint32_t)lane >> 2) * row_bytes + ((uint32_t)lane & 3u) * 16u;
    u32x4 nq = {0u, 0u, 0u, 0u}, ng = nq;
    i32x4 nlab = {0, 0, 0, 0};
    // No branches in here (they would cut the window into pieces): without a next window `on` is false, the
    // descriptors are empty and nothing is fetched.
    // One descriptor per tensor and window (`ask`); the 16 rows of a pass are an offset on top of the lane's own.
    size_t next_q = ((size_t)bw * L * p.ldq + (size_t)h * kHeadDim) * 2u, next_g = ((size_t)bw * L * p.ldg + (size_t)h * kHeadDim) * 2u;
    const size_t step_q = (size_t)gm.G * L * p.ldq * 2u, step_g = (size_t)gm.G * L * p.ldg * 2u;
    u32x4 from_k, from_v;
    auto ask = [&](bool on) {
        from_k = lds_source((const char*)p.k + next_q, on ? tile_bytes : 0u);
        from_v = lds_source((const char*)p.v + next_q, on ? tile_bytes : 0u);
    };
    auto request_slab = [&](uint32_t buf, int t) {  // 16 rows of K and V: block W t + wave
        // a wave beyond the last block moves that one too
        const uint32_t blk = NB % W == 0 || wave + t * W < (uint32_t)NB ? wave + t * W : (uint32_t)NB - 1u;
        const uint32_t to = lds_offset(lds) + buf * (2 * SLAB * 16) + blk * 1024u;
        const uint32_t off = off_slab + here(16u * blk * row_bytes);
        load_to_lds(from_k, off, to);
        load_to_lds(from_v, off, to + SLAB * 16);
    };
    auto request_rest = [&](uint32_t w, bool on) {
        nq = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc((const char*)p.q + next_q, on ? tile_bytes : 0u), off_q, 0, 0);
        ng = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc((const char*)p.d_o + next_g, on ? tile_bytes_g : 0u), off_g, 0, 0);
        if (PW)  // wave 0's are parked; tokens beyond L lie outside the descriptor: label 0
            nlab = load_i32x4(make_rsrc(p.labels + (size_t)(w % (uint32_t)p.nW) * L, on && wave == 0 ? (uint32_t)L * 4u : 0u), (uint32_t)tid * 16u);
    };
    auto park_labels = [&](uint32_t buf) {
        if (PW && tid < ROWS / 4) reinterpret_cast<i32x4*>(llab + buf * ROWS)[tid] = nlab;
    };
    const uint32_t end = (uint32_t)p.N, step = gm.G;
    if (bw < end) {  // in flight while the additive term is fetched
        ask(true);
#pragma unroll
        for (int t = 0; t < PASSES; ++t) request_slab(0u, t);
        request_rest(bw, true);
    }
    next_q += step_q, next_g += step_g;
    f32x4 add[NB];
    if (BM) {  // through the second buffer, which nothing has been requested into yet
        static_assert(W * kFillPatch <= 2 * SLAB * 16, "the buffer holds the waves' patches");
        const BiasSrc rb = bias_of_head(p, h);
        // rows beyond L (and the whole block of an idle wave) fall outside the descriptors: zeros
        const MaskSrc msk = PW ? MaskSrc{make_rsrc(nullptr, 0), 0.f, false} : mask_of_window(p, bw);
        fill_rows_patch<NB>(add, rb, msk, active ? (uint32_t)(16 * qb) : (uint32_t)L, (uint32_t)L, kLog2e,
                            reinterpret_cast<char*>(lds + 2 * SLAB) + wave * kFillPatch, lane);
        __syncthreads();
    }
    for (uint32_t i = (uint32_t)(4 * L + tid); i < SLAB; i += 64u * W) {  // rows L .. ROWS - 1 of the four slabs
        const uint4 z = {0u, 0u, 0u, 0u};
        lds[i] = lds[SLAB + i] = lds[2 * SLAB + i] = lds[3 * SLAB + i] = z;
    }
    const float mv = p.mask_value * kLog2e;
    park_labels(0u);
    lds_loads_done();
    __syncthreads();

    uint32_t buf = 0u;
    for (uint32_t w = bw; w < end; w += step, buf ^= 1u) {
        const uint4* const lk = lds + buf * (2 * SLAB);
        const uint4* const lv = lk + SLAB;
        const bf16x8 qop = as_bf16x8(nq), gop = as_bf16x8(ng);
        const bool has_next = w + step < end;
        ask(has_next);
        float M, nd;
        u32x2 lo, hi;
        if (active) {
            f32x4 s[NB];
            const int* const lab = llab + buf * ROWS;
            const AddendRegsLabels<NB> with_labels = {add, lab, PW ? lab[16 * qb + n] : 0, mv, g};
            // all K operands are asked for at once (they are as large as the scores that replace them), and the
            // products run two blocks ahead of the vector work on them
            float m = -INFINITY;
            bf16x8 ok[NB];
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) ok[jb] = __builtin_bit_cast(bf16x8, lk[opd + 16 * jb * STRIDE]);
#pragma unroll
            for (int jb = 0; jb < NB + 2; ++jb) {
                if (jb < NB) s[jb] = mfma_bf16(ok[jb], qop, zero);
                if (jb >= 2) {
                    const int c = jb - 2;
                    const f32x4 t = PW ? with_labels.block(c) : (BM ? add[c] : zero);
#pragma unroll
                    for (int r = 0; r < 4; ++r) s[c][r] = BM ? fmaf(s[c][r], sl2, t[r]) : s[c][r] * sl2;
                    pad_and_max<NB>(s[c], c, L, g, m);
                }
                if (jb & 1) __builtin_amdgcn_sched_barrier(0);
            }
            rows_block<NB, rows_tight(NB, PW)>(s, m, gop, lk, lv, opd, trs, minus_one, p.scale, M, nd, lo, hi, [&](int i) {
                // the next window's loads one pair at a time: issued in one go they queue at the CU's address unit
                // and hold the wave up
#pragma unroll
                for (int t = 0; t < PASSES; ++t)
                    if (i == 2 * t) request_slab(buf ^ 1u, t);
                if (i == 3) request_rest(w + step, has_next);
            });
        } else {  // an idle wave moves its share all the same
#pragma unroll
            for (int t = 0; t < PASSES; ++t) request_slab(buf ^ 1u, t);
        }
        // The next window's slabs are in LDS before this wave passes the barrier; the
        // wait stands in front of the stores, so that it does not wait for those.
        next_q += step_q, next_g += step_g;
        lds_loads_done();
        park_labels(buf ^ 1u);
        if (active) {
            const size_t tile_d = ((size_t)w * L * p.ldd + (size_t)h * kHeadDim) * 2u;
            // A row beyond L leaves what takes it out of every sum over the queries (its probabilities are zeros), whatever
            // its own scores were: with labels and a mask value of -inf they may be NaN.  (Selects, not a branch, which
            // would cut the window into pieces: 1 % of it.  The kernel below reads dense masks alone, zeros beyond L.)
            const bool pad = 16 * qb + n >= L;
            store_stats<NB>(p, tile_d, row_d, qb, n, g, BM && pad ? INFINITY : M, BM && pad ? 0.f : nd);
            store_rows(cell, lo, hi, make_rsrc((char*)p.dq + tile_d, tile_bytes_d), qb, row_d, lane);
        }
        __syncthreads();  // the next window is in place, and every wave is done with this one's buffer
    }
}

// The rows kernel for dense masks whose period no G is a multiple of: 4 (NB <= 10) or 8 waves walk the query blocks
// of a head, and rows of (bias + mask) are fetched for every window.  A lane needs 4 consecutive keys of one query
// row and neighbouring lanes sit in different rows, which the memory pipeline serves a lane at a time; so the wave
// copies 16 rows x 64 columns at a time with row-contiguous 16-byte loads into a private LDS patch and picks its
// values from there.
constexpr int stream_waves(int nb) { return nb <= 10 ? 4 : 8; }
constexpr uint32_t kPatchRow = 68;  // 64 floats + 4 of padding

template <int NB>
constexpr size_t stream_lds() {
    return (size_t)4 * 16 * NB * kLargeStride * 16 + (size_t)stream_waves(NB) * 16 * kPatchRow * 4;
}

template <int NB, bool HB>
__global__ void __launch_bounds__(64 * stream_waves(NB)) bwd_bf16_rows_stream_kernel(BwdArgs p, LargeGeom gm) {
    constexpr int W = stream_waves(NB);
    constexpr int ROWS = 16 * NB;
    constexpr int PASSES = (ROWS + 16 * W - 1) / (16 * W);
    constexpr uint32_t STRIDE = kLargeStride, SROW = STRIDE * 8, SG = kPatchRow;
    extern __shared__ __attribute__((aligned(16))) uint4 lds[];  // slabs [K][V][Q][dO], each [ROWS][STRIDE]; one patch per wave
    const int tid = threadIdx.x, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lb = xcd_logical_block(blockIdx.x, gm.xcd_q, gm.xcd_r);  // heads of a window: one XCD
    const uint32_t h = lb % gm.heads, bw = lb / gm.heads;
    const int L = p.L;
    const uint32_t row_bytes = (uint32_t)p.ldq * 2u, row_g = (uint32_t)p.ldg * 2u, row_d = (uint32_t)p.ldd * 2u;
    const float sl2 = p.scale * kLog2e;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    uint4* const lk = lds;
    uint4* const lv = lds + ROWS * STRIDE;
    uint4* const lq = lds + 2 * ROWS * STRIDE;
    uint4* const lg = lds + 3 * ROWS * STRIDE;
    float* const patch = reinterpret_cast<float*>(lds + 4 * ROWS * STRIDE) + wave * (16 * SG);
    const uint32_t ll = (uint32_t)L * L * 4u;
    const float* const bias32 = static_cast<const float*>(p.bias);
    const uint32_t srow = (uint32_t)tid >> 2, scol = (uint32_t)tid & 3u;
    const uint32_t tile_bytes = (uint32_t)(L - 1) * row_bytes + 2u * kHeadDim;
    const uint32_t tile_bytes_g = (uint32_t)(L - 1) * row_g + 2u * kHeadDim;
    const uint32_t tile_bytes_d = (uint32_t)(L - 1) * row_d + 2u * kHeadDim;
    const uint32_t trs = (4u * g + (n >> 2)) * SROW + 4u * (n & 3);
    const uint32_t opd = (uint32_t)n * STRIDE + g;

    // The slabs of the next window are requested into registers by every wave right before its last stores of the
    // current one -- the big temporaries are dead by then --, and parked between the two barriers between windows.
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
        // through the window on behalf of the path on which no request happens
#pragma unroll
        for (int t = 0; t < PASSES; ++t) pk[t] = pv[t] = pq[t] = pg[t] = u32x4{0u, 0u, 0u, 0u};

        for (int qb = (int)wave; qb < NB; qb += W) {
            const bf16x8 qop = __builtin_bit_cast(bf16x8, lq[opd + 16 * qb * STRIDE]);
            const bf16x8 gop = __builtin_bit_cast(bf16x8, lg[opd + 16 * qb * STRIDE]);
            // rows 16 qb .. 16 qb + 15 of (bias + mask), 64 columns at a time: lane -> (row 4t + lane / 16,
            // columns 4 (lane % 16) ..), 256 contiguous bytes per 16 lanes; rows beyond L lie outside the
            // descriptors and read as zero, columns beyond L are overwritten with -inf later.  The first
            // patch is requested before the products are formed, each further one a patch ahead.
            const uint32_t prow = (uint32_t)lane >> 4, pcol = 4u * ((uint32_t)lane & 15u);
            constexpr int CH = (NB + 3) / 4;
            f32x4 tb[2][4], tm[2][4];
            const uint32_t qrow = (uint32_t)(16 * qb) * L * 4u;  // < ll: the block starts inside the tile
            const __amdgpu_buffer_rsrc_t rbq =
                HB ? make_rsrc(bias32 + (size_t)h * L * L + (size_t)16 * qb * L, ll - qrow) : make_rsrc(nullptr, 0);
            const __amdgpu_buffer_rsrc_t rmq =
                make_rsrc(p.mask + (size_t)(w % (uint32_t)p.nW) * L * L + (size_t)16 * qb * L, ll - qrow);
            auto request_patch = [&](int ch, int slot) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint32_t off = ((uint32_t)(4 * t + prow) * L + pcol) * 4u + 256u * ch;
                    if (HB) tb[slot][t] = load_f32x4(rbq, off);
                    tm[slot][t] = load_f32x4(rmq, off);
                }
            };
            request_patch(0, 0);
            f32x4 s[NB];
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
                s[jb] = mfma_bf16(__builtin_bit_cast(bf16x8, lk[opd + 16 * jb * STRIDE]), qop, zero);
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) {
                const int cur = ch & 1;
                if (ch + 1 < CH) request_patch(ch + 1, cur ^ 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    *reinterpret_cast<f32x4*>(patch + (4 * t + prow) * SG + pcol) = (HB ? tb[cur][t] + tm[cur][t] : tm[cur][t]) * kLog2e;
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
            float M, nd;
            float m = -INFINITY;
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) pad_and_max<NB>(s[jb], jb, L, g, m);
            u32x2 lo, hi;
            // in the tight form: the longer pipeline gives up to 1 % from 145 tokens on, but 97 tokens take 75.6 us with it, 72.5 without
            rows_block<NB, true>(s, m, gop, lk, lv, opd, trs, bf16x4{0, 0, 0, 0}, p.scale, M, nd, lo, hi, [](int) {});
            if (has_next && qb + W >= NB) request(w + gm.G);  // the wave's last block of this window
            store_stats<NB>(p, tile_d, row_d, qb, n, g, M, nd);
            store_rows(reinterpret_cast<char*>(patch), lo, hi, make_rsrc((char*)p.dq + tile_d, tile_bytes_d), qb, row_d, lane);
        }
        __syncthreads();
        if (has_next) park();
    }
}

// ------------------------------------------------------------------ keys kernel
// At most 4 waves per workgroup (one per SIMD), of which a CU holds two: while one loads or waits at a barrier the
// other computes.  Only Q and dO (all rows) go through LDS; the wave takes the K and V rows of its key block straight
// from global memory.  With DB the dBias accumulator is L x L fp32 per head (256 KB at L = 256), half of a CU's
// register file, spread over the waves of the head's workgroups; the sums are written out once, in register order, as
// one of G partial sums per head, and the reduce kernel adds the slots in a fixed order.
enum { kTermNone = 0,    // no additive term
       kTermKept = 1,    // (bias + mask) * log2e of all queries and the wave's keys in registers, G a multiple of the period
       kTermLabels = 2,  // bias * log2e in registers, the mask from the labels of each window
       kTermStream = 3,  // a dense mask read for every window, and the bias too where the registers are needed for dBias
       kTermStreamMask = 4 };  // a dense mask alone, read for every window

template <int NB>
constexpr size_t keys_lds() {  // two buffers of: Q, dO slabs; then two of: M, -delta, labels; the waves' output cells
    return (size_t)2 * 2 * 16 * NB * kLargeStride * 16 + (size_t)2 * 3 * 16 * NB * 4 + (size_t)keys_waves(NB) * 16 * 80;
}

// Waves per SIMD: two at least; more said for 65 to 80 tokens, where a workgroup is small and the compiler takes a few registers too many.
// Four against three there: no term, dBias, 2048 windows of 65 tokens, 3 heads 67.9 us against 75.6, labels per window without dBias 70.2
// against 87.3.  Three against two: dense mask per window, dBias 91.8 against 94.7.  Three elsewhere only spill: 100 tokens, mask alone per
// window 70.8 against 67.8, 161 tokens, no term 53.5 against 45.8, 81 tokens, labels per window 112 against 69.
constexpr int keys_per_simd(int nb, int term, bool db) { return nb > 5 ? 2 : term == kTermNone || !db ? 4 : 3; }

template <int NB, int TERM, bool DB>
__global__ void __launch_bounds__(64 * keys_waves(NB), keys_per_simd(NB, TERM, DB)) bwd_bf16_keys_kernel(BwdArgs p, LargeGeom gm) {
    constexpr bool KEEP = TERM == kTermKept || TERM == kTermLabels;
    constexpr bool STREAM = TERM == kTermStream || TERM == kTermStreamMask;
    constexpr bool PW = TERM == kTermLabels;
    constexpr bool KEEPB = TERM == kTermStream && NB <= 12;  // the bias in registers all the same
    constexpr bool HB = TERM == kTermStream && !KEEPB;
    // The block during which the next window's rows and statistics are requested: late, while they wait they take registers,
    // but ahead of the loads of a term that is read for every window.  At 65 to 80 tokens the last one is the third: there the last but
    // two would be the first half (bias without dBias 63.8 us against 78.6; labels per window with dBias the other way round, 91.6
    // against 85.9), and 225 to 256 tokens with labels per window have few registers (55.4 against 56.1).
    constexpr int REST_AT = STREAM ? NB / 2 : (NB == 5 && !(PW && DB)) || (NB >= 15 && PW) ? NB - 1 : NB - 3;
    // The products of the lower parts with those of the upper ones, not a block later: fewer registers (65 tokens, bias without dBias 63.8 us
    // against 78.1; mask per window at 97 to 112 tokens 70.8 against 72.7, elsewhere -1 to +1 %).
    constexpr bool EARLY = NB == 5 || STREAM;
    constexpr uint32_t PARTS = (uint32_t)keys_parts(NB);
    constexpr int W = keys_waves(NB);
    constexpr int ROWS = 16 * NB;
    constexpr int PASSES = (ROWS + 16 * W - 1) / (16 * W);
    constexpr uint32_t STRIDE = kLargeStride, SROW = STRIDE * 8;
    extern __shared__ __attribute__((aligned(16))) uint4 lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the parts of a head and the heads of a window are neighbours in the logical order: one XCD
    const uint32_t lb = xcd_logical_block(blockIdx.x, gm.xcd_q, gm.xcd_r);
    const uint32_t part = lb % PARTS, h = (lb / PARTS) % gm.heads, bw = lb / (PARTS * gm.heads);
    const int jb = (int)(part + PARTS * wave);  // this wave's key block
    const bool active = jb < NB;                // wave-uniform
    const int L = p.L;
    const uint32_t row_bytes = (uint32_t)p.ldq * 2u, row_g = (uint32_t)p.ldg * 2u, row_d = (uint32_t)p.ldd * 2u;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const float sl2 = p.scale * kLog2e;
    const bf16x4 minus_one = minus_identity(g, n);

    // two buffers: window w is computed out of one while the slabs of w + G are on their way into the other
    constexpr uint32_t SLAB = ROWS * STRIDE;                              // in uint4
    constexpr uint32_t ST = 3 * ROWS;                                     // M, -delta, labels of a window, in dwords
    float* const stats = reinterpret_cast<float*>(lds + 4 * SLAB);
    char* const cell = reinterpret_cast<char*>(stats + 2 * ST) + wave * (16 * 80);

    const uint32_t ll = (uint32_t)L * L * 4u;
    const float* const bias32 = static_cast<const float*>(p.bias);
    const uint32_t tile_bytes = (uint32_t)(L - 1) * row_bytes + 2u * kHeadDim;
    const uint32_t tile_bytes_g = (uint32_t)(L - 1) * row_g + 2u * kHeadDim;
    const uint32_t tile_bytes_d = (uint32_t)(L - 1) * row_d + 2u * kHeadDim;
    const uint32_t trs = (4u * g + (n >> 2)) * SROW + 4u * (n & 3);
    const uint32_t opd = (uint32_t)n * STRIDE + g;

    f32x4 dbacc[NB];  // dS summed over the windows: queries 16 qb + 4g + r, key 16 jb + n
    if (DB) {
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) dbacc[qb] = zero;
    }

    // The Q and dO slabs of the next window go straight from memory into the other LDS buffer (no registers, no LDS
    // writes), requested over the first half of a window's blocks; its statistics (wave 0: M, wave 1: -delta, 16 bytes per lane), its
    // labels and the wave's own K and V rows are requested at block REST_AT and wait in registers.  Rows beyond L are never loaded: zeros from the start.
    static_assert(W >= 3, "wave 2 fetches the labels");
    const uint32_t off_q = ((uint32_t)lane >> 2) * row_bytes + ((uint32_t)lane & 3u) * 16u, off_g = ((uint32_t)lane >> 2) * row_g + ((uint32_t)lane & 3u) * 16u;
    static_assert(4 * SLAB * 16 <= 65536, "direct loads reach the first 64 KB");
    u32x4 pst = {0u, 0u, 0u, 0u}, pk = pst, pv = pst;
    // No branches in here (they would cut the block loop into pieces): without a next window `on` is false, the
    // descriptors are empty and nothing is fetched.
    // One descriptor per tensor and window (`ask`); the 16 rows of a pass are an offset on top of the lane's own.
    // The windows are walked from the last to the first: what the rows kernel has touched last is in the 256 MB cache (16 x 16
    // windows 321.2 -> 317.4 us, 14 x 14 93.5 -> 92.5).
    uint32_t left = bw < (uint32_t)p.N ? ((uint32_t)p.N - bw + gm.G - 1u) / gm.G : 0u;
    uint32_t w = bw + (left - 1u) * gm.G;
    size_t next_q = ((size_t)w * L * p.ldq + (size_t)h * kHeadDim) * 2u, next_g = ((size_t)w * L * p.ldg + (size_t)h * kHeadDim) * 2u;
    size_t next_d = ((size_t)w * L * p.ldd + (size_t)h * kHeadDim) * 2u;
    const size_t step_q = (size_t)gm.G * L * p.ldq * 2u, step_g = (size_t)gm.G * L * p.ldg * 2u, step_d = (size_t)gm.G * L * p.ldd * 2u;
    u32x4 from_q, from_g;
    auto ask = [&](bool on) {
        from_q = lds_source((const char*)p.q + next_q, on ? tile_bytes : 0u);
        from_g = lds_source((const char*)p.d_o + next_g, on ? tile_bytes_g : 0u);
    };
    auto request_slab = [&](uint32_t buf, int t) {  // 16 rows of Q and dO: block W t + wave
        // a wave beyond the last block moves that one too
        const uint32_t blk = NB % W == 0 || wave + t * W < (uint32_t)NB ? wave + t * W : (uint32_t)NB - 1u;
        const uint32_t to = lds_offset(lds) + buf * (2 * SLAB * 16) + blk * 1024u;
        load_to_lds(from_q, off_q + here(16u * blk * row_bytes), to);
        load_to_lds(from_g, off_g + here(16u * blk * row_g), to + SLAB * 16);
    };
    auto request_rest = [&](uint32_t w, bool on) {
        // waves 0, 1: floats 4 lane .. 4 lane + 3 of M resp. -delta, i.e. row 16 part + lane / 4 of the head's slice
        // of dV resp. dK; wave 2 with PW: labels 4 lane .. 4 lane + 3 (0 beyond L)
        const char* src = (wave == 0 ? static_cast<const char*>(p.dv) : static_cast<const char*>(p.dk)) + next_d;
        uint32_t bytes = wave < 2 ? (16u * PARTS - 1u) * row_d + 64u : 0u;
        if (PW) {
            const char* const lab = reinterpret_cast<const char*>(p.labels + (size_t)(w % (uint32_t)p.nW) * L);
            src = wave == 2 ? lab : src;
            bytes = wave == 2 ? (uint32_t)L * 4u : bytes;
        }
        const uint32_t l = (uint32_t)lane;
        const uint32_t off_st = wave < 2 ? (16u * part + (l >> 2)) * row_d + 16u * (l & 3u) : 16u * l;
        pst = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(src, on ? bytes : 0u), off_st, 0, 0);
        // the wave's own K and V rows as operands: row 16 jb + n, channels 8g .. 8g + 7
        const uint32_t off = (16u * jb + (l & 15u)) * row_bytes + 16u * (l >> 4), own = on ? tile_bytes : 0u;
        pk = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc((const char*)p.k + next_q, own), off, 0, 0);
        pv = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc((const char*)p.v + next_q, own), off, 0, 0);
    };
    auto park = [&](uint32_t buf) {
        // M, -delta and labels lie one behind the other: ROWS / 4 = 4 NB <= 64 units of 16 bytes each
        if (wave < (PW ? 3u : 2u) && lane < ROWS / 4) reinterpret_cast<u32x4*>(stats + buf * ST + wave * ROWS)[lane] = pst;
    };
    if (left > 0) {  // in flight while the additive term is fetched
        ask(true);
#pragma unroll
        for (int t = 0; t < PASSES; ++t) request_slab(0u, t);
        request_rest(w, true);
    }
    next_q -= step_q, next_g -= step_g, next_d -= step_d;
    f32x4 add[NB];  // (bias + mask) * log2e, resp. bias * log2e, in the layout of dbacc
    if (KEEP || KEEPB) {
        const MaskSrc msk = PW || KEEPB ? MaskSrc{make_rsrc(nullptr, 0), 0.f, false} : mask_of_window(p, bw);
        // rows beyond L lie outside the descriptors: zeros.  A key beyond L reads into the next row: what it makes
        // of that stays in its own column of every product, i.e. in rows of dV, dK and columns of dBias beyond L,
        // which the stores and the reduce kernel drop.
        const BiasSrc rb = bias_of_head(p, h);
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) {
            const uint32_t off = ((uint32_t)(16 * qb + 4 * g) * L + 16u * jb + n) * 4u;
            const f32x4 mk = mask_rows4(msk, (uint32_t)(16 * qb + 4 * g), 16u * jb + n, (uint32_t)L);
#pragma unroll
            for (int r = 0; r < 4; ++r) add[qb][r] = (load_f32(rb.r, off + 4u * L * r) + mk[r]) * kLog2e;
        }
    }
    for (uint32_t i = (uint32_t)(4 * L + tid); i < SLAB; i += 64u * W) {  // rows L .. ROWS - 1 of the four slabs
        const uint4 z = {0u, 0u, 0u, 0u};
        lds[i] = lds[SLAB + i] = lds[2 * SLAB + i] = lds[3 * SLAB + i] = z;
    }
    uint32_t aoff[4];  // STREAM: additive term of query 4g + r (of a query block) and this lane's key
#pragma unroll
    for (int r = 0; r < 4; ++r) aoff[r] = ((uint32_t)(4 * g + r) * L + 16u * jb + n) * 4u;
    const float mv = p.mask_value * kLog2e;
    if (left > 0) park(0u);
    lds_loads_done();
    __syncthreads();

    uint32_t buf = 0u;
    for (; left > 0; w -= gm.G, buf ^= 1u, --left) {
        take_turns(left);
        const uint4* const lq = lds + buf * (2 * SLAB);
        const uint4* const lg = lq + SLAB;
        const float* const stM = stats + buf * ST;
        const float* const stD = stM + ROWS;  // -delta
        const int* const llab = reinterpret_cast<const int*>(stD + ROWS);
        const uint16_t* const lg16 = reinterpret_cast<const uint16_t*>(lg) + trs;
        const uint16_t* const lq16 = reinterpret_cast<const uint16_t*>(lq) + trs;
        const size_t tile_d = next_d + step_d;
        const bf16x8 kop = as_bf16x8(pk), vop = as_bf16x8(pv);
        const bool has_next = left > 1;
        ask(has_next);
        u32x2 va = {0u, 0u}, vb = {0u, 0u}, ka = {0u, 0u}, kb = {0u, 0u};  // the wave's 16 rows of dV and dK, packed

        if (active) {
            const int lkey = PW ? llab[16 * jb + n] : 0;
            f32x4 v0 = zero, v1 = zero, k0 = zero, k1 = zero;  // dV, dK [16 jb + n][4g + r] and [..][16 + 4g + r]
            // The products S, dP of a query block are issued one block ahead of the block's vector work, from operands
            // fetched two blocks ahead; what remains of P and dS after their upper parts is made by the matrix core and packed during
            // the next block, and the dV, dK products of a pair of blocks follow in the next two: so every
            // stretch of vector instructions has matrix instructions beside it that do not depend on it.
            bf16x8 oq, og, tg0, tg1, tx0, tx1;
            u32x4 PH = {0u, 0u, 0u, 0u}, SH = PH, PL = PH, SL = PH;  // operands of a pair: upper and lower parts of P and dS
            f32x4 oM[2], oD, sc, dp, rp = zero, rs = zero, ab[2], am[2];
            i32x4 al[2];
            auto fetch_q = [&](int qb) {
                oq = __builtin_bit_cast(bf16x8, lq[opd + 16 * qb * STRIDE]);
                og = __builtin_bit_cast(bf16x8, lg[opd + 16 * qb * STRIDE]);
                oD = *reinterpret_cast<const f32x4*>(stD + 16 * qb + 4 * g);
            };
            auto fetch_m = [&](int qb) {
                oM[qb & 1] = *reinterpret_cast<const f32x4*>(stM + 16 * qb + 4 * g);
                if (PW) al[qb & 1] = *reinterpret_cast<const i32x4*>(llab + 16 * qb + 4 * g);
            };
            auto fetch_term = [&](int qb) {
                // descriptors start at the first row of the query block, so that the 4 lane offsets
                // serve every block; rows beyond L lie outside them
                const uint32_t qrow = (uint32_t)(16 * qb) * L;
                const __amdgpu_buffer_rsrc_t rbq =
                    HB ? make_rsrc(bias32 + (size_t)h * L * L + qrow, ll - 4u * qrow) : make_rsrc(nullptr, 0);
                const __amdgpu_buffer_rsrc_t rmq =
                    make_rsrc(p.mask + (size_t)(w % (uint32_t)p.nW) * L * L + qrow, ll - 4u * qrow);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (HB) ab[qb & 1][r] = load_f32(rbq, aoff[r]);
                    am[qb & 1][r] = load_f32(rmq, aoff[r]);
                }
            };
            auto products = [&]() {
                sc = mfma_bf16(oq, kop, zero);  // <q_i, k_j>, i = 16 qb + 4g + r, j = 16 jb + n
                dp = mfma_bf16(og, vop, oD);  // dP - delta
            };
            auto fetch_t = [&](int qp) {  // dO^T and Q^T of the 32 queries (channel on the lane)
                const bool two = 2 * qp + 1 < NB;
                tg0 = operand_tr(lg16 + (32 * qp) * SROW, 16 * SROW, two);
                tg1 = operand_tr(lg16 + (32 * qp) * SROW + 16, 16 * SROW, two);
                tx0 = operand_tr(lq16 + (32 * qp) * SROW, 16 * SROW, two);
                tx1 = operand_tr(lq16 + (32 * qp) * SROW + 16, 16 * SROW, two);
            };
            auto accumulate = [&](const u32x4& pp, const u32x4& ss) {
                v0 = mfma_bf16(tg0, as_bf16x8(pp), v0);
                v1 = mfma_bf16(tg1, as_bf16x8(pp), v1);
                k0 = mfma_bf16(tx0, as_bf16x8(ss), k0);
                k1 = mfma_bf16(tx1, as_bf16x8(ss), k1);
            };
            auto lower = [&](int u) {  // of block u of a pair
                PL[2 * u] = pack_bf16(rp[0], rp[1]), PL[2 * u + 1] = pack_bf16(rp[2], rp[3]);
                SL[2 * u] = pack_bf16(rs[0], rs[1]), SL[2 * u + 1] = pack_bf16(rs[2], rs[3]);
            };
            fetch_q(0);
            if (STREAM) fetch_term(0);
            products();
            fetch_q(1);
            fetch_m(0);
            if (STREAM) fetch_term(1);
#pragma unroll
            for (int qb = 0; qb < NB; ++qb) {
                const int u = qb & 1;
                __builtin_amdgcn_sched_barrier(0);
                // the next window's loads one pair at a time between the blocks: issued in one go they queue at the
                // CU's address unit and hold the wave up
#pragma unroll
                for (int t = 0; t < PASSES; ++t)
                    if (qb == t * (NB / 2) / PASSES) request_slab(buf ^ 1u, t);
                if (qb == REST_AT) request_rest(w - gm.G, has_next);
                if (EARLY && u == 0 && qb > 0) lower(1);
                if (u == 0 && qb > 0) accumulate(PH, SH);
                if (EARLY ? u == 0 && qb > 0 : u == 1 && qb > 1) accumulate(PL, SL);
                if (u == 1) fetch_t(qb / 2);
                if (qb + 1 < NB) fetch_m(qb + 1);
                if (qb > 0 && !(EARLY && u == 0)) lower(u ^ 1);
                f32x4 pr, ds;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // The score is rounded as in the rows kernel before M leaves it (without a term too, where one fma would make the
                    // exponent): so the probabilities are those that its sums were made of, whatever the size of the scores.
                    float t = 0.f;
                    if (STREAM) t = KEEPB ? fmaf(am[u][r], kLog2e, add[qb][r]) : (HB ? ab[u][r] + am[u][r] : am[u][r]) * kLog2e;
                    else if (TERM != kTermNone) t = PW ? add[qb][r] + (al[u][r] == lkey ? 0.f : mv) : add[qb][r];
                    const float x = fmaf(sc[r], sl2, t) - oM[u][r];
                    pr[r] = __builtin_amdgcn_exp2f(x);
                    ds[r] = pr[r] * dp[r];
                }
                if (DB) dbacc[qb] += ds;
                if (STREAM && qb + 2 < NB) fetch_term(qb + 2);
                PH[2 * u] = pack_bf16(pr[0], pr[1]), PH[2 * u + 1] = pack_bf16(pr[2], pr[3]);
                rp = remainder(minus_one, uint2{PH[2 * u], PH[2 * u + 1]}, pr);
                SH[2 * u] = pack_bf16(ds[0], ds[1]), SH[2 * u + 1] = pack_bf16(ds[2], ds[3]);
                rs = remainder(minus_one, uint2{SH[2 * u], SH[2 * u + 1]}, ds);
                if (qb + 1 < NB) products();
                if (qb + 2 < NB) fetch_q(qb + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (NB % 2 == 1) {
                if (!EARLY) accumulate(PL, SL);  // of the last whole pair
                fetch_t(NB / 2);
                PH[2] = PH[3] = SH[2] = SH[3] = PL[2] = PL[3] = SL[2] = SL[3] = 0u;
            }
            lower((NB - 1) & 1);
            accumulate(PH, SH);
            accumulate(PL, SL);
            va = u32x2{pack_bf16(v0[0], v0[1]), pack_bf16(v0[2], v0[3])};
            vb = u32x2{pack_bf16(v1[0], v1[1]), pack_bf16(v1[2], v1[3])};
            ka = u32x2{pack_bf16(k0[0] * p.scale, k0[1] * p.scale), pack_bf16(k0[2] * p.scale, k0[3] * p.scale)};
            kb = u32x2{pack_bf16(k1[0] * p.scale, k1[1] * p.scale), pack_bf16(k1[2] * p.scale, k1[3] * p.scale)};
        } else {  // an idle wave moves its share all the same
#pragma unroll
            for (int t = 0; t < PASSES; ++t) request_slab(buf ^ 1u, t);
            request_rest(w - gm.G, has_next);
        }
        // The next window's slabs are in LDS before this wave passes the barrier; the wait stands in front of the
        // stores, so that it does not wait for those.
        next_q -= step_q, next_g -= step_g, next_d -= step_d;
        lds_loads_done();
        park(buf ^ 1u);
        if (active) {
            store_rows(cell, va, vb, make_rsrc((char*)p.dv + tile_d, tile_bytes_d), jb, row_d, lane);
            store_rows(cell, ka, kb, make_rsrc((char*)p.dk + tile_d, tile_bytes_d), jb, row_d, lane);
        }
        __syncthreads();  // the next window is in place, and every wave is done with this one's buffer
    }

    // partial sums in register order: [slot][head][jb][qb][lane] float4, element r of lane (g, n) being
    // dS summed over windows for query 16 qb + 4g + r and key 16 jb + n
    if (DB && active) {
        f32x4* dst = reinterpret_cast<f32x4*>(p.partial) + ((size_t)bw * p.heads + h) * (NB * NB * 64) + lane;
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) dst[(jb * NB + qb) * 64] = dbacc[qb];
    }
}

// ------------------------------------------------------------------ launches
}  // namespace

// Workgroups of `fn` one CU holds (LDS and registers decide), asked once per kernel; threads racing
// through the first call ask twice and store the same figure.
hipError_t workgroups_per_cu(const void* fn, unsigned block, size_t lds, std::atomic<int>& once, int& per_cu) {
    const hipError_t e = allow_lds(fn, lds);
    if (e != hipSuccess) return e;
    per_cu = once.load(std::memory_order_relaxed);
    if (per_cu == 0) {
        int nblk = 0;
        const hipError_t q = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nblk, fn, (int)block, lds);
        if (q != hipSuccess) return q;
        per_cu = nblk < 1 ? 1 : nblk;
        once.store(per_cu, std::memory_order_relaxed);
    }
    return hipSuccess;
}

namespace {

LargeGeom large_geom(const BwdArgs& a, int parts, long long G, unsigned& grid) {
    LargeGeom gm;
    gm.heads = (uint32_t)a.heads;
    gm.parts = (uint32_t)parts;
    gm.G = (uint32_t)G;
    grid = gm.G * gm.heads * gm.parts;
    gm.xcd_q = grid / 8u;
    gm.xcd_r = grid % 8u;
    return gm;
}

// Window positions walked in parallel, `resident` = as many as the chip holds at once.  Without a mask period: those,
// at most one per window.  With one, a workgroup that keeps its additive term needs a multiple of it: the largest
// that is resident, unless the rounding leaves so much idle that the form that takes the mask per window, and has no
// period to keep to, is faster (0 is returned for that one).  Per window it takes 1.35 times as long with a dense mask.
// With labels only 1.08 times, but while a call keeps its term its results are those of the dense mask bit for bit, which
// is not given up for less than a quarter of the time (kept : per window, us, labels: 125 windows of 256 tokens, 3 heads,
// period 25 53.9 : 42.8; 270 of 196, 9 heads, period 9 219 : 172; where nothing is rounded away, 1448 of 225, 2 heads,
// period 4, dBias 218 : 238; 1512 of 256, 1 head, period 12 137 : 150).  For a dense mask with a longer period (`rounds`)
// more than are resident at once, in several rounds, as long as the cost in windows -- rounds times (windows per workgroup
// + about one and a half for fetching the term) -- stays below that of the kernels that read the mask per window (L = 256:
// 210 against 154 us and 283 against 185).  `most`: an upper limit (the dBias slots).
long long walk_slots(long long resident, long long most, long long N, long long period, bool dense, bool rounds) {
    if (resident < 1) resident = 1;
    long long G = resident < most ? resident : most;
    if (G > N) G = N;
    const long long fit = G / period * period;
    const double whole = (double)((N + G - 1) / G);  // windows per workgroup with nothing rounded away
    if (fit > 0) {
        const double kept = (double)((N + fit - 1) / fit);
        return kept > (dense ? 1.35 * whole + 1.0 : 1.3 * whole + 0.5) ? 0 : fit;
    }
    if (!rounds) return 0;
    const double stream = 1.35 * whole;
    long long best = 0;
    double best_cost = stream;
    for (long long c = period; c <= N && c <= most && c <= 16 * resident; c += period) {
        const double cost = (double)((c + resident - 1) / resident) * ((double)(N / c + (N % c != 0)) + 1.5);
        if (cost < best_cost) best_cost = cost, best = c;
    }
    return best;
}

template <int NB, bool BM, bool PW>
hipError_t launch_rows(const BwdArgs& a, long long period, hipStream_t st, bool& fits) {
    const void* fn = reinterpret_cast<const void*>(&bwd_bf16_rows_kernel<NB, BM, PW>);
    constexpr unsigned block = 64u * rows_waves(NB);
    static std::atomic<int> once{0};
    int per_cu = 1;
    const hipError_t e = workgroups_per_cu(fn, block, rows_lds<NB>(), once, per_cu);
    if (e != hipSuccess) return e;
    const long long G = walk_slots((long long)cu_count() * per_cu / ((long long)a.heads * rows_parts(NB)), a.N, a.N, period, a.mask != nullptr, a.mask != nullptr);
    fits = G > 0;
    if (!fits) return hipSuccess;
    unsigned grid;
    const LargeGeom gm = large_geom(a, rows_parts(NB), G, grid);
    hipLaunchKernelGGL((bwd_bf16_rows_kernel<NB, BM, PW>), dim3(grid), dim3(block), rows_lds<NB>(), st, a, gm);
    return hipGetLastError();
}

template <int NB, bool HB>
hipError_t launch_rows_stream(const BwdArgs& a, hipStream_t st) {
    const void* fn = reinterpret_cast<const void*>(&bwd_bf16_rows_stream_kernel<NB, HB>);
    constexpr unsigned block = 64u * stream_waves(NB);
    static std::atomic<int> once{0};
    int per_cu = 1;
    const hipError_t e = workgroups_per_cu(fn, block, stream_lds<NB>(), once, per_cu);
    if (e != hipSuccess) return e;
    unsigned grid;
    const LargeGeom gm = large_geom(a, 1, walk_slots((long long)cu_count() * per_cu / a.heads, a.N, a.N, 1, false, false), grid);
    hipLaunchKernelGGL((bwd_bf16_rows_stream_kernel<NB, HB>), dim3(grid), dim3(block), stream_lds<NB>(), st, a, gm);
    return hipGetLastError();
}

// window slots of the keys kernel (0: none fits the period)
template <int NB, int TERM, bool DB>
hipError_t keys_slots(const BwdArgs& a, long long period, bool rounds, long long& G) {
    static std::atomic<int> once{0};
    int per_cu = 1;
    const hipError_t e = workgroups_per_cu(reinterpret_cast<const void*>(&bwd_bf16_keys_kernel<NB, TERM, DB>), 64u * keys_waves(NB), keys_lds<NB>(), once, per_cu);
    const long long resident = (long long)cu_count() * per_cu / ((long long)a.heads * keys_parts(NB));
    const long long most = DB ? a.slots : a.N;  // the workspace holds a.slots partial sums per head
    G = walk_slots(resident, most, a.N, period, a.mask != nullptr, rounds);
    return e;
}
// dK, dV and, with DB, the dBias partial sums and their reduction
template <int NB, int TERM, bool DB>
hipError_t launch_keys(const BwdArgs& a, long long period, hipStream_t st, bool& fits) {
    long long G = 0;
    const hipError_t e = keys_slots<NB, TERM, DB>(a, period, a.mask != nullptr, G);
    fits = G > 0;
    if (e != hipSuccess || !fits) return e;
    unsigned grid;
    const LargeGeom gm = large_geom(a, keys_parts(NB), G, grid);
    hipLaunchKernelGGL((bwd_bf16_keys_kernel<NB, TERM, DB>), dim3(grid), dim3(64u * keys_waves(NB)), keys_lds<NB>(), st, a, gm);
    const hipError_t l = hipGetLastError();
    if (!DB || l != hipSuccess) return l;
    BwdArgs r = a;
    r.slots = (int)G;
    return launch_dbias_reduce(r, st, true);
}

// The additive term stays in registers where the number of window positions in flight can be a multiple of the mask
// period (1 without a mask).  Beyond that labels let the kernels form the mask of each window, and a dense mask is
// read per window.  The two kernels decide for themselves: they hold different numbers of workgroups.  Calls without
// dBias go to the fused kernel where it is the faster one; with a dense mask whose period the resident workgroups cannot
// hold it is (nW = 64, 8 heads, 2048 tiles, pair : fused, us: L = 144 95.7 : 85.6, L = 196 181 : 165, L = 256 214 : 210),
// but for the smallest windows while launching more than the resident ones will do (L = 81: 35.7 : 39.5).
template <int NB>
hipError_t launch_large_nb(const BwdArgs& a, hipStream_t st) {
    if (a.bias && a.bias_bf16) return hipErrorInvalidValue;  // the caller hands over an fp32 copy
    const bool bm = a.bias || has_mask(a);
    const long long period = mask_period(a);
    if (!a.dbias) {
        bool forced = !bm, taken = false;
        long long G = 1;  // of the keys kernel as it would run
        if (bm) {
            hipError_t q = keys_slots<NB, kTermKept, false>(a, period, a.mask && NB <= 6, G);
            forced = a.mask && G == 0;
            if (q == hipSuccess && G == 0) q = keys_slots<NB, kTermKept, false>(a, 1, false, G);
            if (q != hipSuccess) return q;
        }
        const hipError_t e = launch_backward_bf16_fused(a, st, forced, (a.N + G - 1) / G, taken);
        if (e != hipSuccess || taken) return e;
    }
    bool fits = false;
    hipError_t e = bm ? launch_rows<NB, true, false>(a, period, st, fits) : launch_rows<NB, false, false>(a, 1, st, fits);
    if (e == hipSuccess && !fits) {
        if (a.labels) e = launch_rows<NB, true, true>(a, 1, st, fits);
        else e = a.bias ? launch_rows_stream<NB, true>(a, st) : launch_rows_stream<NB, false>(a, st);
    }
    if (e != hipSuccess) return e;
    if (!a.dbias) {
        e = launch_keys<NB, kTermKept, false>(a, period, st, fits);
        if (e == hipSuccess && !fits) e = a.labels ? launch_keys<NB, kTermLabels, false>(a, 1, st, fits) : hipErrorInvalidValue;
        return e;
    }
    e = bm ? launch_keys<NB, kTermKept, true>(a, period, st, fits) : launch_keys<NB, kTermNone, true>(a, 1, st, fits);
    if (e == hipSuccess && !fits) {
        if (a.labels) e = launch_keys<NB, kTermLabels, true>(a, 1, st, fits);
        else e = a.bias ? launch_keys<NB, kTermStream, true>(a, 1, st, fits) : launch_keys<NB, kTermStreamMask, true>(a, 1, st, fits);
    }
    return e;
}

}  // namespace

// Slots of dBias partial sums for large windows: one resident workgroup of the keys kernel per CU
// when its slabs fill most of the LDS (more than 10 blocks of 16 rows), two otherwise
int backward_large_slots(long long N, int heads, int L) {
    long long G = (L > 160 ? 1 : 2) * cu_count() / heads;
    if (G < 1) G = 1;
    return (int)(G > N ? N : G);
}

hipError_t launch_backward_bf16_large(const BwdArgs& a, hipStream_t s) {
    switch ((a.L + 15) / 16) {
        case 5: return launch_large_nb<5>(a, s);
        case 6: return launch_large_nb<6>(a, s);
        case 7: return launch_large_nb<7>(a, s);
        case 8: return launch_large_nb<8>(a, s);
        case 9: return launch_large_nb<9>(a, s);
        case 10: return launch_large_nb<10>(a, s);
        case 11: return launch_large_nb<11>(a, s);
        case 12: return launch_large_nb<12>(a, s);
        case 13: return launch_large_nb<13>(a, s);
        case 14: return launch_large_nb<14>(a, s);
        case 15: return launch_large_nb<15>(a, s);
        case 16: return launch_large_nb<16>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fwa
