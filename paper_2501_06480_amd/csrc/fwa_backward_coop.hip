// Cooperative backward kernel (paper Algorithm 2) for L <= 64: one wave per 16-row block of a
// (window, head) tile (NB = ceil(L / 16) waves), several heads per workgroup, persistent over windows.
//
// One wave per tile would need the whole register file and run two waves per SIMD (built first: twice as
// slow).  Here the tile is split:
//
//   phase A, wave qb (16 queries, "query on the lane"):
//       S^T = K Q^T, softmax, dP^T = V dO^T, delta, dS          (K, V rows read from LDS)
//       dQ rows of its block (contraction over keys: dS is already the B operand)
//       dBias rows of its block, accumulated in registers across windows
//       P and dS rows of its block, as hi + lo bf16, written row-major into LDS tiles
//   phase B, wave jb (16 keys):
//       dV, dK rows of its block = contraction over all queries of P resp. dS with dO^T resp.
//       Q^T.  The operands with the queries on the k-slots come out of LDS through the
//       transposing read ds_read_b64_tr_b16: the P/dS tiles with the key on the lane, the
//       dO/Q slabs (and the K slab for dQ in phase A) with the channel on the lane.
//
// The workgroup loads the Q, K, V, dO slabs of its heads (whole 128-byte lines per row) with
// coalesced 16-byte loads into LDS once per window and requests the next window's slabs before
// computing.  A workgroup keeps its heads and walks the windows bw, bw + G, ...; G is a
// multiple of nW, so (bias[h] + mask[bw % nW]) * log2e is loaded once, into registers.
#include "fwa_device.h"
#include "fwa_internal.h"
#include "fwa_softmax.h"

#include <algorithm>

namespace fwa {
namespace {

constexpr int kCoopMaxHeads = 3;  // heads per workgroup
// Compiled for 12 waves per CU at every NB, though below 49 tokens a workgroup has fewer
constexpr int kCoopBoundThreads = 64 * 4 * kCoopMaxHeads;
// Waves per SIMD the registers leave room for (NB = 1, 2: at most 128)
constexpr int coop_waves_per_simd(int nb) { return nb <= 2 ? 4 : 3; }

struct CoopGeom {
    FastDiv groups;         // workgroups per window position
    FastDiv lanes_per_row;  // 4 * heads_per_block
    uint32_t heads_per_block;
    uint32_t stride;        // slab row in 16-byte units
    uint32_t G;             // window positions walked in parallel (= dBias slots)
    uint32_t xcd_remap, xcd_q, xcd_r;
};

// Mask tiles in LDS of the form that fetches one per window (PW == 2 below): two up to 48 tokens.
__host__ __device__ constexpr uint32_t coop_mask_tiles(int nb) { return nb <= 3 ? 2u : 1u; }

// KT < 4 promises that only the first KT of a lane's 4 columns in the last key block can be real
// (L <= 16 (NB - 1) + KT, e.g. KT = 1 for L = 49): the others are zero without any arithmetic.
// PW ("per window"): G is no multiple of the mask's period.  The registers then hold bias * log2e alone.
// PW = 1, labels: those of a window travel with its slabs into LDS and phase A forms the mask per score
// (AddendRegsLabels).  PW = 2, a dense mask: the tile of a window is fetched into LDS during the window before (L > 48:
// during its phase B, there is room for one tile), straight from memory and in whole lines (AddendRegsDense; every lane
// loading the values of its own row, 16 bytes of a line each, took 93 us instead of 53 below).  Stage 1 of two 800 x 1333 images (2784
// windows, 3 heads, bias, mask of 1392 windows, dBias): 53 us with the reduction, 52 as labels; a kernel with one
// wave per tile that such calls took before, 102.
template <int NB, bool BM, bool DB, int KT, int PW>
__global__ void __launch_bounds__(kCoopBoundThreads) bwd_bf16_coop_kernel(BwdArgs p, CoopGeom gm) {
    constexpr int NB2 = (NB + 1) / 2;
    constexpr int ROWS = 16 * NB;
    extern __shared__ __attribute__((aligned(16))) uint4 lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t hl = wv / (uint32_t)NB;      // head inside the workgroup
    const int role = (int)(wv % (uint32_t)NB);  // query block in phase A, key block in phase B
    // workgroups that share 128-byte lines (head groups of one window) are neighbours in the logical
    // order; when a group is not made of whole lines the order is mapped so that they share an XCD
    const uint32_t lb = gm.xcd_remap ? xcd_logical_block(blockIdx.x, gm.xcd_q, gm.xcd_r) : blockIdx.x;
    const uint32_t bw = fastdiv(lb, gm.groups);
    const uint32_t hg = lb - bw * gm.groups.d;
    const uint32_t hpb = gm.heads_per_block;
    const uint32_t h = hg * hpb + hl;
    const int L = p.L;
    // token rows are p.ldq (q, k, v), p.ldg (d_o), p.ldd (dq, dk, dv) elements apart; window w starts at row w L
    const uint32_t row_bytes = (uint32_t)p.ldq * 2u, row_g = (uint32_t)p.ldg * 2u, row_d = (uint32_t)p.ldd * 2u;
    const uint32_t stride = gm.stride;  // slab row stride in 16-byte units
    const float sl2 = p.scale * kLog2e;
    // Always true.  Below 49 tokens the branches on it keep the compiler from mixing the phases (NB = 3 with dBias: 142
    // registers, 168 and 16 spills without them).
    const bool active = NB == 4 || h < (uint32_t)p.heads;

    // LDS: (PW == 2) one or two mask tiles; slabs [K][V][Q][dO], each [ROWS][stride] uint4; then per head four bf16 tiles.
    constexpr bool TWO = coop_mask_tiles(NB) == 2;  // PW == 2: room for the next window's tile beside the current one
    constexpr bool TURN = KT == 4;  // row lengths that are multiples of 16 are not among those of a smaller KT
    const uint32_t mask_units = PW == 2 ? mask_tile_bytes((uint32_t)L) / 16u : 0u;
    uint4* const lmask = lds;
    uint4* const lk = lds + coop_mask_tiles(NB) * mask_units;
    uint4* const lv = lk + ROWS * stride;
    uint4* const lq = lk + 2 * ROWS * stride;
    uint4* const lg = lk + 3 * ROWS * stride;
    // P_hi, P_lo, dS_hi, dS_lo tiles of this head: [ROWS][64] bf16.  A row is 16 units of 4 keys; unit
    // (block b, quarter c) of row i sits at unit (b ^ (i & 3), c ^ ((i >> 2) & 3)): the 16 lanes of a
    // write (16 rows, one unit each) and of a transposing read (4 rows x 4 units) then touch 16
    // different units, i.e. every bank once.
    constexpr uint32_t XS = 64, XT = ROWS * XS;
    uint16_t* const ex = reinterpret_cast<uint16_t*>(lk + 4 * ROWS * stride) + (size_t)hl * (4 * XT);
    // PW == 1: the labels of the window in LDS, behind the tiles of all heads
    int* const llab = reinterpret_cast<int*>(reinterpret_cast<uint16_t*>(lk + 4 * ROWS * stride) + (size_t)hpb * (4 * XT));
    const uint32_t srow = stride * 8u;  // slab row stride in bf16 elements
    // transposing-read base of this lane inside a slab (channel on the lane) and inside a tile
    const uint32_t trs = (4u * g + (n >> 2)) * srow + 32u * hl + 4u * (n & 3);
    // transposing read of key block jb = role: row 4g + (n >> 2) (+ 16, 32, ...: same low row bits)
    const uint32_t trx = (4u * g + (n >> 2)) * XS + ((((uint32_t)role) ^ (uint32_t)(n >> 2)) << 4) + ((((uint32_t)n & 3u) ^ (uint32_t)g) << 2);
    const uint32_t opd = (uint32_t)n * stride + 4u * hl + g;  // operand of row block b: slab[opd + 16 b stride]

    f32x4 dbacc[NB];
#pragma unroll
    for (int jb = 0; jb < NB; ++jb) dbacc[jb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    // Remainders of the splits of P and dS from the matrix core: above 49 tokens, where they save 2 to 7 % (128 windows of 64 tokens, 32
    // heads, labels 48.8 -> 46.0 us), and at 49 with dBias (Swin-T stage 1 with bias and mask 127.7 -> 126.7).  At 49 without dBias the last
    // block holds one key, and they cost 1 to 6 % (4096 windows, 12 heads, bias 248 -> 263); fewer blocks would lose a wave per SIMD.
    constexpr bool MATRIX = NB == 4 && (KT == 4 || DB);
    [[maybe_unused]] const bf16x4 minus_one = minus_identity(g, n);

    // slab movement: thread -> (row, 16-byte column); 4 hpb threads per row and 64 NB hpb threads: one pass covers
    // the slab.  (rip < ROWS holds for every thread; without the branches on it the compiler mixes the stores with what
    // stands around them: Swin-T stage 1 with bias, mask and dBias 128.4 -> 129.6 us.)
    const uint32_t rip = fastdiv((uint32_t)tid, gm.lanes_per_row);
    const uint32_t col = (uint32_t)tid - rip * gm.lanes_per_row.d;
    const uint32_t slab_bytes = (uint32_t)(L - 1) * row_bytes + hpb * 2u * kHeadDim;
    const uint32_t slab_bytes_g = (uint32_t)(L - 1) * row_g + hpb * 2u * kHeadDim;
    const uint32_t goff = rip * row_bytes + col * 16u;
    const uint32_t goff_g = rip * row_g + col * 16u;
    const uint32_t loff = rip * stride + col;
    u32x4 pk, pv, pq, pg;
    i32x4 plab = {0, 0, 0, 0};  // PW == 1: labels 4 tid .. 4 tid + 3 of the requested window (0 beyond L)
    auto request = [&](uint32_t w) {
        const size_t slab = ((size_t)w * L * p.ldq + (size_t)hg * hpb * kHeadDim) * 2u;
        const size_t slab_g = ((size_t)w * L * p.ldg + (size_t)hg * hpb * kHeadDim) * 2u;
        // rows beyond L lie outside the descriptors and arrive as zeros
        pk = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc((const char*)p.k + slab, slab_bytes), goff, 0, 0);
        pv = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc((const char*)p.v + slab, slab_bytes), goff, 0, 0);
        pq = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc((const char*)p.q + slab, slab_bytes), goff, 0, 0);
        pg = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc((const char*)p.d_o + slab_g, slab_bytes_g), goff_g, 0, 0);
        if (PW == 1 && wv == 0) plab = load_i32x4(make_rsrc(p.labels + (size_t)(w % (uint32_t)p.nW) * L, (uint32_t)L * 4u), (uint32_t)tid * 16u);
    };
    auto park = [&]() {
        if (rip < (uint32_t)ROWS) {
            lk[loff] = __builtin_bit_cast(uint4, pk);
            lv[loff] = __builtin_bit_cast(uint4, pv);
            lq[loff] = __builtin_bit_cast(uint4, pq);
            lg[loff] = __builtin_bit_cast(uint4, pg);
        }
        if (PW == 1 && tid < ROWS / 4) reinterpret_cast<i32x4*>(llab)[tid] = plab;
    };
    if (bw < (uint32_t)p.N) request(bw);  // in flight while the additive term is fetched
    // additive score term of this wave's query rows, in registers (see the file comment)
    f32x4 add[NB];
    if (BM) {
        const BiasSrc rb = bias_of_head(p, h);
        const MaskSrc msk = PW ? MaskSrc{make_rsrc(nullptr, 0), 0.f, false} : mask_of_window(p, bw);
        bool filled = false;
        if constexpr (NB == 4) {
            filled = fill_in_lines<NB>(p, false);
            if (filled) {
                f32x4 one[1][NB];
                const uint32_t rows0[1] = {(uint32_t)(16 * role)};
                // through the exchange tiles of the head, which are not in use yet (the barrier that opens the first
                // window stands between these reads and their first writes)
                static_assert(NB * rows_fill_bytes<NB>() <= 4 * XT * 2, "the tiles hold the waves' stretches");
                fill_rows_staged<1, NB>(one, rb, msk, rows0, (uint32_t)L, kLog2e, reinterpret_cast<char*>(ex) + role * rows_fill_bytes<NB>(), lane);
#pragma unroll
                for (int jb = 0; jb < NB; ++jb) add[jb] = one[0][jb];
            }
        }
        if (!filled) {
            const uint32_t i = (uint32_t)(16 * role + n);
            addend_at(rb, mask_of_row(msk, i, (uint32_t)L), i, 4u * g, (uint32_t)L).fill(add, kLog2e);
        }
    }
    const float mv = 16 * role + n < L ? p.mask_value * kLog2e : 0.f;
    auto request_mask = [&](uint32_t w, uint32_t tile) { request_mask_tile<TURN>(p, w, lds_offset(lmask) + tile * mask_units * 16u, wv, NB * hpb, (uint32_t)lane); };
    // this lane's query row of the mask tile; rows beyond L stay inside it (their results are dropped)
    const int mask_i = 16 * role + n < L ? 16 * role + n : L - 1;
    const float* const mask_row = reinterpret_cast<const float*>(lmask) + mask_i * L;
    const uint32_t mask_turn = TURN ? mask_tile_turn((uint32_t)mask_i, (uint32_t)L) : 0u;
    if (PW == 2 && bw < (uint32_t)p.N) request_mask(bw, 0u);
    if (bw < (uint32_t)p.N) park();
    if (PW == 2) lds_loads_done();

    const uint32_t tile_bytes = (uint32_t)(L - 1) * row_d + 2u * kHeadDim;  // of an output tile
    const uint32_t off_half = (uint32_t)n * row_d + 8u * g;  // channels 4g..4g+3 of row n (+32 B: 16+4g..)

    // The next window's slabs are requested at the top of an iteration and parked in LDS at its
    // end, i.e. always with this iteration's output stores younger than them in the memory queue:
    // the wait in front of the LDS writes then counts those stores out instead of waiting for them
    // (at the top of the loop the compiler has to assume the worst of both ways in).  The request
    // stands behind the barrier, not in front of it: a wave that is held up while it issues its
    // loads (the 48 wave-level loads of a workgroup queue at the CU's one address unit) then holds
    // up nobody else (stage 1: 135 -> 128 us, stage 2: 75 -> 70; spreading the four loads of a
    // thread over the stages of phase A adds nothing to that).
    uint32_t mtile = 0u;  // PW == 2: the mask tile of the window
    for (uint32_t w = bw; w < (uint32_t)p.N; w += gm.G) {
        const bool has_next = w + gm.G < (uint32_t)p.N;
        __syncthreads();
        if (PW == 2 && TWO && has_next) request_mask(w + gm.G, mtile ^ 1u);
        if (has_next) request(w + gm.G);  // in flight while this window is computed

        const size_t tile = ((size_t)w * L * p.ldd + (size_t)h * kHeadDim) * 2u;
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        u32x2 dq_lo = {0u, 0u}, dq_hi = {0u, 0u};
        // ---------------- phase A: query block `role` ----------------
        if (active) {
            const int qb = role;
            const bf16x8 qop = __builtin_bit_cast(bf16x8, lq[opd + 16 * qb * stride]);
            const bf16x8 gop = __builtin_bit_cast(bf16x8, lg[opd + 16 * qb * stride]);
            f32x4 s[NB], dp[NB];
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
                s[jb] = mfma_bf16(__builtin_bit_cast(bf16x8, lk[opd + 16 * jb * stride]), qop, zero);
                dp[jb] = mfma_bf16(__builtin_bit_cast(bf16x8, lv[opd + 16 * jb * stride]), gop, zero);
            }
            // softmax of the block's rows: s <- exp(score - rowmax), inv = 1 / rowsum
            float inv;
            if (BM && PW == 2) {
                const AddendRegsDense<NB> addend = {add, mask_row + mtile * mask_units * 4u, mask_turn, (uint32_t)g};
                inv = softmax_block<NB, true, AddendRegsDense<NB>, KT>(s, sl2, addend, L, g);
            } else if (BM && PW == 1) {
                const AddendRegsLabels<NB> addend = {add, llab, llab[16 * qb + n], mv, g};
                inv = softmax_block<NB, true, AddendRegsLabels<NB>, KT>(s, sl2, addend, L, g);
            } else if (BM) {
                const AddendRegs<NB> addend = {add};
                inv = softmax_block<NB, true, AddendRegs<NB>, KT>(s, sl2, addend, L, g);
            } else {
                inv = softmax_block<NB, false, AddendNone, KT>(s, sl2, AddendNone{}, L, g);
            }
            float delta = 0.f;
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                for (int r = 0; r < (jb == NB - 1 ? KT : 4); ++r) {
                    s[jb][r] *= inv;  // P
                    delta = fmaf(s[jb][r], dp[jb][r], delta);
                }
            delta = sum_over_g(delta);
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    dp[jb][r] = (jb == NB - 1 && r >= KT) ? 0.f : s[jb][r] * (dp[jb][r] - delta);  // dS
                if (DB) dbacc[jb] += dp[jb];
            }
            // hi + lo bf16 parts of P and dS: rows of this block into the LDS tiles for phase B.  MATRIX: what remains after the upper
            // parts comes from the matrix core, for all blocks before the first is packed.
            bf16x4 p_hi[NB], ds_hi[NB], ds_lo[NB];
            if constexpr (MATRIX) {
#pragma unroll
                for (int jb = 0; jb < NB; ++jb) {
                    p_hi[jb] = packed4(s[jb]);
                    s[jb] = remainder(minus_one, p_hi[jb], s[jb]);
                    ds_hi[jb] = packed4(dp[jb]);
                    dp[jb] = remainder(minus_one, ds_hi[jb], dp[jb]);
                }
            }
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
                bf16x4 p_lo;
                if constexpr (MATRIX) {
                    p_lo = packed4(s[jb]), ds_lo[jb] = packed4(dp[jb]);
                } else {
                    split_hi_lo(s[jb], p_hi[jb], p_lo);
                    split_hi_lo(dp[jb], ds_hi[jb], ds_lo[jb]);
                }
                uint16_t* cell = ex + (16 * qb + n) * XS + ((jb ^ (n & 3)) << 4) + ((g ^ ((n >> 2) & 3)) << 2);
                *reinterpret_cast<uint2*>(cell + 0 * XT) = __builtin_bit_cast(uint2, p_hi[jb]);
                *reinterpret_cast<uint2*>(cell + 1 * XT) = __builtin_bit_cast(uint2, p_lo);
                *reinterpret_cast<uint2*>(cell + 2 * XT) = __builtin_bit_cast(uint2, ds_hi[jb]);
                *reinterpret_cast<uint2*>(cell + 3 * XT) = __builtin_bit_cast(uint2, ds_lo[jb]);
            }
            // dQ^T = K^T dS^T over pairs of key blocks; K^T (channels 0..15 / 16..31 on the lane)
            // straight from the K slab
            f32x4 q0 = zero, q1 = zero;  // dQ[16 qb + n][4g + r], dQ[16 qb + n][16 + 4g + r]
            const uint16_t* lk16 = reinterpret_cast<const uint16_t*>(lk) + trs;
#pragma unroll
            for (int kp = 0; kp < NB2; ++kp) {
                const bool two = 2 * kp + 1 < NB;
                const int j1 = two ? 2 * kp + 1 : 0;
                const bf16x8 k0 = operand_tr(lk16 + (32 * kp) * srow, 16 * srow, two);
                const bf16x8 k1 = operand_tr(lk16 + (32 * kp) * srow + 16, 16 * srow, two);
                const uint2 h0 = __builtin_bit_cast(uint2, ds_hi[2 * kp]), l0 = __builtin_bit_cast(uint2, ds_lo[2 * kp]);
                uint2 h1 = {0u, 0u}, l1 = {0u, 0u};
                if (two) {
                    h1 = __builtin_bit_cast(uint2, ds_hi[j1]);
                    l1 = __builtin_bit_cast(uint2, ds_lo[j1]);
                }
                const bf16x8 dh = as_bf16x8(u32x4{h0.x, h0.y, h1.x, h1.y}), dl = as_bf16x8(u32x4{l0.x, l0.y, l1.x, l1.y});
                q0 = mfma_bf16(k0, dh, q0);
                q1 = mfma_bf16(k1, dh, q1);
                q0 = mfma_bf16(k0, dl, q0);
                q1 = mfma_bf16(k1, dl, q1);
            }
            dq_lo = u32x2{pack_bf16(q0[0] * p.scale, q0[1] * p.scale), pack_bf16(q0[2] * p.scale, q0[3] * p.scale)};
            dq_hi = u32x2{pack_bf16(q1[0] * p.scale, q1[1] * p.scale), pack_bf16(q1[2] * p.scale, q1[3] * p.scale)};
        }
        __syncthreads();
        // ---------------- phase B: key block `role` ----------------
        if (active) {
            {   // the dQ rows of phase A leave behind the barrier
                const __amdgpu_buffer_rsrc_t rdq = make_rsrc((char*)p.dq + tile, tile_bytes);
                __builtin_amdgcn_raw_buffer_store_b64(dq_lo, rdq, off_half + 16 * role * row_d, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b64(dq_hi, rdq, off_half + 32 + 16 * role * row_d, 0, 0);
            }
        }
        if (PW == 2 && !TWO && has_next) request_mask(w + gm.G, 0u);  // every wave has left phase A, the tile's only reader
        if (active) {
            const int jb = role;
            f32x4 v0 = zero, v1 = zero, k0 = zero, k1 = zero;  // dV, dK [16 jb + n][4g + r] and [..][16 + 4g + r]
            const uint16_t* lg16 = reinterpret_cast<const uint16_t*>(lg) + trs;
            const uint16_t* lq16 = reinterpret_cast<const uint16_t*>(lq) + trs;
            const uint16_t* xt = ex + trx;
#pragma unroll
            for (int qp = 0; qp < NB2; ++qp) {
                const bool two = 2 * qp + 1 < NB;
                // dO^T and Q^T of the 32 queries (channel on the lane), P and dS of the same
                // queries (key on the lane)
                const bf16x8 g0 = operand_tr(lg16 + (32 * qp) * srow, 16 * srow, two);
                const bf16x8 g1 = operand_tr(lg16 + (32 * qp) * srow + 16, 16 * srow, two);
                const bf16x8 x0 = operand_tr(lq16 + (32 * qp) * srow, 16 * srow, two);
                const bf16x8 x1 = operand_tr(lq16 + (32 * qp) * srow + 16, 16 * srow, two);
                const bf16x8 ph = operand_tr(xt + 0 * XT + (32 * qp) * XS, 16 * XS, two);
                const bf16x8 pl = operand_tr(xt + 1 * XT + (32 * qp) * XS, 16 * XS, two);
                const bf16x8 sh = operand_tr(xt + 2 * XT + (32 * qp) * XS, 16 * XS, two);
                const bf16x8 sl = operand_tr(xt + 3 * XT + (32 * qp) * XS, 16 * XS, two);
                v0 = mfma_bf16(g0, ph, v0);
                v1 = mfma_bf16(g1, ph, v1);
                k0 = mfma_bf16(x0, sh, k0);
                k1 = mfma_bf16(x1, sh, k1);
                v0 = mfma_bf16(g0, pl, v0);
                v1 = mfma_bf16(g1, pl, v1);
                k0 = mfma_bf16(x0, sl, k0);
                k1 = mfma_bf16(x1, sl, k1);
            }
            const u32x2 va = {pack_bf16(v0[0], v0[1]), pack_bf16(v0[2], v0[3])};
            const u32x2 vb = {pack_bf16(v1[0], v1[1]), pack_bf16(v1[2], v1[3])};
            const u32x2 ka = {pack_bf16(k0[0] * p.scale, k0[1] * p.scale), pack_bf16(k0[2] * p.scale, k0[3] * p.scale)};
            const u32x2 kb = {pack_bf16(k1[0] * p.scale, k1[1] * p.scale), pack_bf16(k1[2] * p.scale, k1[3] * p.scale)};
            // The rows leave through the K and V slabs, which nothing reads in phase B (only this wave
            // touches its head's 64-byte slice of its 16 rows), and from there as whole rows.
            u32x2* const rowv = reinterpret_cast<u32x2*>(lv + (16 * jb + n) * stride + 4 * hl);
            u32x2* const rowk = reinterpret_cast<u32x2*>(lk + (16 * jb + n) * stride + 4 * hl);
            rowv[g] = va;
            rowv[4 + g] = vb;
            rowk[g] = ka;
            rowk[4 + g] = kb;
        }
        __syncthreads();  // dK, dV rows complete; slabs and exchange area are rewritten by the next window
        if (rip < (uint32_t)ROWS) {  // 16 bytes per lane, whole rows; rows beyond L are dropped by the range check
            const size_t slab_d = ((size_t)w * L * p.ldd + (size_t)hg * hpb * kHeadDim) * 2u;
            const uint32_t slab_bytes_d = (uint32_t)(L - 1) * row_d + hpb * 2u * kHeadDim;
            const uint32_t goff_d = rip * row_d + col * 16u;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, lk[loff]), make_rsrc((char*)p.dk + slab_d, slab_bytes_d), goff_d, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, lv[loff]), make_rsrc((char*)p.dv + slab_d, slab_bytes_d), goff_d, 0, 0);
        }
        if (PW == 2) {  // the mask tile has landed; the two stores above are younger and not waited for
            wait_vmem<2>();
            if (TWO) mtile ^= 1u;
        }
        if (has_next) park();  // each thread overwrites the slab cells it has just read out
    }

    if (DB) {
        // partial sums in register order: [slot][head][qb][jb][lane] float4 -- contiguous 16-byte stores
        f32x4* dst = reinterpret_cast<f32x4*>(p.partial) + ((size_t)bw * p.heads + h) * (NB * NB * 64) + lane;
#pragma unroll
        for (int jb = 0; jb < NB; ++jb) {
            // What lies beyond L is never read.  Above 48 tokens it is not stored either (38 % at 49); below, asking costs more than it saves
            // (8192 windows of 25 tokens, 8 heads 171 -> 176 us).
            if (NB < 4 || (16 * role + n < L && (jb < NB - 1 || 16 * jb + 4 * g < L))) dst[(role * NB + jb) * 64] = dbacc[jb];
        }
    }
}

// LDS of a workgroup: slabs, exchange tiles, and the mask tiles or the labels of a window where those come per window
size_t coop_lds(int nb, int hpb, int L, bool mask_tiles, bool labels, uint32_t& stride) {
    const size_t rows = (size_t)16 * nb;
    const size_t tiles = hpb * 4 * rows * 64 * 2 + (mask_tiles ? coop_mask_tiles(nb) * mask_tile_bytes((uint32_t)L) : 0) + (labels ? rows * 4 : 0);
    // one unit of padding per slab row, but where a dense mask tile per window takes its place: at 3 heads and
    // L = 56 .. 64 the workgroup then fills the 160 KB of LDS exactly
    stride = 4 * rows * (4 * hpb + 1) * 16 + tiles <= 160 * 1024 ? 4u * (uint32_t)hpb + 1u : 4u * (uint32_t)hpb;
    return 4 * rows * stride * 16 + tiles;
}

template <int NB, bool BM, bool DB, int KT, int PW>
hipError_t launch_coop_pw(const BwdArgs& a, const CoopGeom& gm, unsigned grid, unsigned block, size_t lds,
                          hipStream_t st) {
    {
        const hipError_t e = allow_lds(reinterpret_cast<const void*>(&bwd_bf16_coop_kernel<NB, BM, DB, KT, PW>), lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((bwd_bf16_coop_kernel<NB, BM, DB, KT, PW>), dim3(grid), dim3(block), lds, st, a, gm);
    return hipGetLastError();
}

template <int NB, bool BM, bool DB, int KT>
hipError_t launch_coop_kt(const BwdArgs& a, const CoopGeom& gm, unsigned grid, unsigned block, size_t lds,
                          hipStream_t st) {
    if constexpr (BM) {
        if (a.per_window)
            return a.labels ? launch_coop_pw<NB, true, DB, KT, 1>(a, gm, grid, block, lds, st)
                            : launch_coop_pw<NB, true, DB, KT, 2>(a, gm, grid, block, lds, st);
    }
    return launch_coop_pw<NB, BM, DB, KT, 0>(a, gm, grid, block, lds, st);
}

template <int NB, bool BM, bool DB>
hipError_t launch_coop_one(const BwdArgs& a, const CoopGeom& gm, unsigned grid, unsigned block, size_t lds,
                           hipStream_t st) {
    // a single column in the last key block (L = 16 (NB - 1) + 1: the 7 x 7 window): the trimmed variant
    if (a.L == 16 * (NB - 1) + 1 && NB > 1) return launch_coop_kt<NB, BM, DB, 1>(a, gm, grid, block, lds, st);
    return launch_coop_kt<NB, BM, DB, 4>(a, gm, grid, block, lds, st);
}

template <int NB>
hipError_t launch_coop_nb(const BwdArgs& a, int hpb, hipStream_t st) {
    CoopGeom gm;
    const uint32_t groups = (uint32_t)(a.heads / hpb);
    gm.groups = make_fastdiv(groups);
    gm.lanes_per_row = make_fastdiv(4u * (uint32_t)hpb);
    gm.heads_per_block = (uint32_t)hpb;
    gm.G = (uint32_t)a.slots;
    const unsigned grid = gm.G * groups, block = 64u * NB * (unsigned)hpb;
    const size_t lds = coop_lds(NB, hpb, a.L, a.per_window && a.mask, a.per_window && a.labels, gm.stride);
    gm.xcd_remap = (hpb % 2 == 1 && groups > 1) ? 1u : 0u;
    gm.xcd_q = grid / 8u;
    gm.xcd_r = grid % 8u;
    const bool bm = a.bias || has_mask(a), db = a.dbias != nullptr;
    if (bm)
        return db ? launch_coop_one<NB, true, true>(a, gm, grid, block, lds, st)
                  : launch_coop_one<NB, true, false>(a, gm, grid, block, lds, st);
    return db ? launch_coop_one<NB, false, true>(a, gm, grid, block, lds, st)
              : launch_coop_one<NB, false, false>(a, gm, grid, block, lds, st);
}

}  // namespace

// Heads per workgroup of the cooperative kernel: all of them when the row has at most 3 (the
// slab is then whole rows: full 128-byte lines in and out).  Beyond that, groups of 2 (whole
// lines) or 3 heads with one workgroup per CU, or single heads with three 4-wave workgroups per
// CU that run their phases independently but fetch and store 64-byte halves of lines.  Measured,
// backward with dBias: 4, 8, 16, 32 heads in pairs are 16-18 % faster than singly (Swin-B stages
// 1-4); 6 and 12 heads in threes 14 % and 8 % faster at 8192 and 2048 windows (Swin-L stages 1, 2)
// but 2-5 % slower at 512 and 128 windows (Swin-T stages 3, 4), where a workgroup meets too few
// windows to make up for its longer set-up: threes from 16 windows per workgroup on.  With 48
// heads (Swin-L stage 4, 128 windows) threes are 8 % faster already at 8 windows per workgroup
// (24 heads at 256 windows: no difference either way).
int coop_heads_per_block(int heads, long long N) {
    if (heads <= kCoopMaxHeads) return heads;
    if (heads % 3 == 0)   // windows per workgroup = N / (compute units / (heads / 3))
        return (N * heads >= 16LL * 3 * cu_count() || (heads >= 48 && N * heads >= 8LL * 3 * cu_count())) ? 3 : 1;
    return heads % 2 == 0 ? 2 : 1;
}

// Window positions walked in parallel: about one workgroup per CU (LDS allows no more), a
// multiple of nW so that every workgroup keeps one mask tile; 0 = the kernel does not apply.
int coop_slots(long long N, int heads, int nW) {
    const int hpb = coop_heads_per_block(heads, N);
    if (hpb == 0 || nW < 1) return 0;
    const int groups = heads / hpb;
    const int per_cu = hpb == 3 ? 1 : (hpb == 2 ? 1 : 3);
    long long G = ((long long)cu_count() * per_cu / groups) / nW * nW;
    if (G > N) G = N / nW * nW;
    if (G < nW || G <= 0) return 0;
    return (int)G;
}

// Heads per workgroup where the masks come per window: a dense tile at 33 to 48 tokens leaves a CU room for one workgroup of
// two or three heads, but for three of one (2142 windows of 36 tokens, 4 heads, dBias: pairs 50.7 us, singly 46).
int coop_window_heads_per_block(int heads, long long N, int nb, bool dense) {
    return dense && nb == 3 ? 1 : coop_heads_per_block(heads, N);
}

// Window positions walked in parallel where the masks come per window, which leave no period to keep to.  From 33 tokens
// on as above, as far as LDS holds the workgroups.  Below, LDS and registers hold more (one workgroup of a pair of heads
// per CU left most of it idle): 4125 windows of 16 tokens, 8 heads, dense masks 87 us at one per CU, 40 at as many as fit;
// 2600 of 25, 7 heads, labels, dBias 47.8 : 43.6.  With dBias every workgroup adds to what the reduction reads: more only
// while each has eight windows, and not for the dense masks of single heads at 17 to 32 tokens (1600 windows, 6 heads
// 30.8 us at three per CU, 35.0 at five).
int coop_window_slots(long long N, int heads, int L, bool dense, bool dbias) {
    const int nb = (L + 15) / 16, hpb = coop_window_heads_per_block(heads, N, nb, dense);
    uint32_t stride;
    const long long lds = (long long)coop_lds(nb, hpb, L, dense, !dense, stride);
    const long long fit = std::max(1LL, std::min(160 * 1024 / lds, (long long)(4 * coop_waves_per_simd(nb) / (nb * hpb))));
    const int groups = heads / hpb;
    long long G = cu_count() * std::min(fit, hpb == 1 ? 3LL : 1LL) / groups;
    if (nb == 1 || (nb == 2 && !(dense && dbias && hpb == 1)))
        G = std::max(G, std::min(cu_count() * fit / groups, dbias ? N / 8 : N));
    return (int)std::max(1LL, std::min(G, N));
}

hipError_t launch_backward_bf16_coop(const BwdArgs& a, hipStream_t s) {
    const int nb = (a.L + 15) / 16;
    const int hpb = a.per_window ? coop_window_heads_per_block(a.heads, a.N, nb, a.mask != nullptr) : coop_heads_per_block(a.heads, a.N);
    switch (nb) {
        case 1: return launch_coop_nb<1>(a, hpb, s);
        case 2: return launch_coop_nb<2>(a, hpb, s);
        case 3: return launch_coop_nb<3>(a, hpb, s);
        case 4: return launch_coop_nb<4>(a, hpb, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fwa
