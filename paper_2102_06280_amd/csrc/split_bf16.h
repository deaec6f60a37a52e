// fp32 products on the bf16 matrix instructions, without giving up any of the 24 significant bits.
//
// A finite fp32 value is the exact sum of three bf16 values: its upper 16 bits (high), the remainder rounded to
// bf16 (middle), and what is left (low; at most 8 significant bits, so it is exact as well).  The product of two
// split values has nine partial products; the six kept here,
//   low * high + high * low + middle * middle + middle * high + high * middle + high * high,
// leave out terms below 2^-24 of the product that have no preferred sign.  Every partial product of two bf16 values is exact in
// fp32 and the matrix instruction accumulates in fp32.  v_mfma_f32_32x32x16_bf16 multiplies 16 times as
// many values per cycle as v_mfma_f32_32x32x2_f32 does, so six of them per 16-wide step have 2.7 times the rate: a
// register-resident loop reaches 312 TFLOP/s of fp32 products against 155 (212 to 246 when both operands are split
// in the loop as well).  The result is closer to the exact sum than the fp32 instruction's, because an accumulator is
// rounded 6 times per 16 terms instead of 8 times, and 5 of the 6 additions are small ones: relative error against
// 64 bits 1.1e-7 / 2.4e-7 / 4.3e-7 / 7.0e-7 at 64 / 256 / 800 / 2048 terms, against 1.4e-7 / 2.9e-7 / 5.1e-7 /
// 8.1e-7 (normally distributed operands; positive weights give the same figures).  With all small partial products of a sum
// first, or in an accumulator of their own, the large ones are rounded once per 16 terms: a third of that error again.
//
// An operand that is not finite makes the middle value NaN, and with it every small partial product it enters: an infinity
// does not survive as one.  It does among the large ones, which is why their sum decides (add_small).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace split_bf16 {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Eight values as three planes of eight bf16.
struct planes {
    u32x4 h, m, l;
};

__device__ __forceinline__ uint32_t bits(float v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ float value(uint32_t v) { return __builtin_bit_cast(float, v); }
// the upper halves of a (low 16 bits of the result) and b
__device__ __forceinline__ uint32_t upper(float a, float b) { return __builtin_amdgcn_perm(bits(b), bits(a), 0x07060302u); }

// Two values at a time: 11 vector instructions.
__device__ __forceinline__ void split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l)
{
    h = upper(a, b);
    a -= value(bits(a) & 0xffff0000u);
    b -= value(bits(b) & 0xffff0000u);
    const bf16x2 r = {(__bf16)a, (__bf16)b};          // to nearest
    m = __builtin_bit_cast(uint32_t, r);
    a -= value(m << 16);
    b -= value(m & 0xffff0000u);
    l = upper(a, b);
}

__device__ __forceinline__ planes split8(const float (&x)[8])
{
    planes p;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t h, m, l;
        split2(x[2 * q], x[2 * q + 1], h, m, l);
        p.h[q] = h;
        p.m[q] = m;
        p.l[q] = l;
    }
    return p;
}

__device__ __forceinline__ bf16x8 frag(const u32x4 &v) { return __builtin_bit_cast(bf16x8, v); }

// large + small += a b over 16 terms (32 x 32 outputs).  Lane l holds row (or column) l % 32 of the operand and the terms 8 (l / 32) ..
// + 7 of the step: any assignment of terms to lanes that is the same for both operands gives the same sums.  The large partial
// products, of 16 bits each, have an accumulator of their own, which is rounded once per 16 terms and for a few terms hardly at all;
// the sum of the two (the caller's) is two to three times closer to the exact one than a single accumulator (9e-8 at
// 256 terms, 1.6e-7 at 800); also two shorter chains of dependent instructions.
__device__ __forceinline__ void mma32(const planes &a, const planes &b, f32x16 &large, f32x16 &small)
{
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.l), frag(b.h), small, 0, 0, 0);
    large = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.h), frag(b.h), large, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.h), frag(b.l), small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.m), frag(b.m), small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.m), frag(b.h), small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.h), frag(b.m), small, 0, 0, 0);
}

// Six partial products (or the five small ones, or the large one) for a block of A x B accumulators, one kind after the other,
// the large one last: consecutive instructions are independent.
template <bool SMALL, bool LARGE, int A, int B>
__device__ __forceinline__ void mma32_block(const planes (&a)[A], const planes (&b)[B], f32x16 (&acc)[A][B])
{
    auto step = [&](u32x4 planes::*pa, u32x4 planes::*pb) {
#pragma unroll
        for (int i = 0; i < A; ++i)
#pragma unroll
            for (int j = 0; j < B; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a[i].*pa), frag(b[j].*pb), acc[i][j], 0, 0, 0);
    };
    if (SMALL) {
        step(&planes::l, &planes::h);
        step(&planes::h, &planes::l);
        step(&planes::m, &planes::m);
        step(&planes::m, &planes::h);
        step(&planes::h, &planes::m);
    }
    if (LARGE) step(&planes::h, &planes::h);
}

// NaN or infinity
__device__ __forceinline__ bool not_finite(float v) { return (bits(v) & 0x7f800000u) == 0x7f800000u; }

// whether any value of an accumulator is NaN or infinite (0 * v is NaN then)
__device__ __forceinline__ bool any_not_finite(const f32x16 &acc)
{
    float t = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) t = fmaf(acc[v], 0.f, t);
    return t != t;
}

// large += small, where large is finite.  The high plane holds an infinity or NaN as what it is and zero as zero, so a large sum
// that is not finite is what fp32 multiply-adds give; the small one is then NaN for reasons of its own (a middle value next to an infinity
// has either sign or is zero).
__device__ __forceinline__ void add_small(f32x16 &large, const f32x16 &small)
{
    if (__any(any_not_finite(large))) {
#pragma unroll
        for (int v = 0; v < 16; ++v) large[v] = not_finite(large[v]) ? large[v] : large[v] + small[v];
    } else {
        large += small;
    }
}

// The same where one accumulator is all there is room for: the small partial products of the whole reduction first, then this, then the
// large ones on top.
__device__ __forceinline__ void drop_not_finite(f32x16 &small)
{
#pragma unroll
    for (int v = 0; v < 16; ++v) small[v] = not_finite(small[v]) ? 0.f : small[v];
}

}  // namespace split_bf16

