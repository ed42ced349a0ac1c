// fp32 values as three bf16 values each, for products on the bf16 matrix instruction with 24 significant bits (see
// fwa_f32_rows.hip).
#pragma once

#include "fwa_device.h"

namespace fwa {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
struct Planes {
    u32x2 h, m, l;  // four values as 3 x 4 bf16
};
// two values -> their packed upper parts; what remains of them is left in a, b (exact)
__device__ __forceinline__ uint32_t take_upper(float& a, float& b, bf16x2 first, bf16x2 second) {
    const uint32_t u = pack_bf16(a, b);
    const bf16x2 h = __builtin_bit_cast(bf16x2, u);
    a = __builtin_amdgcn_fdot2_f32_bf16(h, first, a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(h, second, b, false);
    return u;
}
__device__ __forceinline__ Planes split3(const f32x4& x) {
    uint32_t c0 = 0x0000bf80u, c1 = 0xbf800000u;  // (-1, 0), (0, -1): out of registers, as a literal the compiler takes the first for the inline constant -1.0f, which the instruction reads as (0, -1)
    asm("" : "+s"(c0));
    asm("" : "+s"(c1));
    const bf16x2 first = __builtin_bit_cast(bf16x2, c0), second = __builtin_bit_cast(bf16x2, c1);
    float a = x[0], b = x[1], c = x[2], d = x[3];
    const uint32_t h0 = take_upper(a, b, first, second), h1 = take_upper(c, d, first, second);
    const uint32_t m0 = take_upper(a, b, first, second), m1 = take_upper(c, d, first, second);
    return Planes{u32x2{h0, h1}, u32x2{m0, m1}, u32x2{pack_bf16(a, b), pack_bf16(c, d)}};
}
// The same bits with the remainders from the matrix core (minus_identity, fwa_device.h): six conversions and two matrix instructions
// for four values a lane instead of six and eight dot products, which wait for the matrix core to be idle.  Takes two registers
// more, and an infinity or a NaN spreads to the lanes with the same n: for callers whose tiles with such values go another way.
__device__ __forceinline__ Planes split3(bf16x4 minus_one, const f32x4& x) {
    const bf16x4 h = packed4(x);
    const f32x4 y = remainder(minus_one, h, x);
    const bf16x4 m = packed4(y);
    const bf16x4 l = packed4(remainder(minus_one, m, y));
    return Planes{__builtin_bit_cast(u32x2, h), __builtin_bit_cast(u32x2, m), __builtin_bit_cast(u32x2, l)};
}
struct Operand3 {
    bf16x8 h, m, l;
};
__device__ __forceinline__ Operand3 operand3(const Planes& a, const Planes& b) {
    return Operand3{as_bf16x8(u32x4{a.h.x, a.h.y, b.h.x, b.h.y}), as_bf16x8(u32x4{a.m.x, a.m.y, b.m.x, b.m.y}),
                    as_bf16x8(u32x4{a.l.x, a.l.y, b.l.x, b.l.y})};
}
// the largest magnitude of four values; NaN if one is
__device__ __forceinline__ float largest(float m, const f32x4& x) {
    const float a = x[0], b = x[1], c = x[2], d = x[3];
    asm("v_maximum3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
    asm("v_maximum3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(c), "v"(d));
    return m;
}
// The smallest step of a bf16 is 2^-133 (subnormal ones count: the conversion, the dot product and the matrix instruction take
// and give them), so the thirds of a value below 2^-110 lose bits, 2^-134 at most.  Times kLift every fp32 value has exact
// thirds, subnormal ones too.  Multiplying by it and by its inverse (kDrop: for a product of two) is exact.
constexpr int kLiftBits = 16;
constexpr float kLift = 0x1p16f, kDrop = 0x1p-32f;
// Lifted values of which the largest is `top` (below 2^43 as they were) have products whose sums of up to 256 stay finite in every
// part.  Beyond that a product of fp32 values overflows as a whole, to one infinity, but its parts to infinities of both signs.  A
// NaN does not fit either: it would spread to the value it shares a register with.
__device__ __forceinline__ bool fits_lifted(float top) { return top < 0x1p59f; }
// The five small ones of the six products (the largest, h h', is the caller's), smallest first.
__device__ __forceinline__ f32x4 small_products(const Operand3& a, const Operand3& b, f32x4 acc) {
    acc = mfma_bf16(a.l, b.h, acc);
    acc = mfma_bf16(a.h, b.l, acc);
    acc = mfma_bf16(a.m, b.m, acc);
    acc = mfma_bf16(a.m, b.h, acc);
    return mfma_bf16(a.h, b.m, acc);
}

}  // namespace fwa
