// fp32 products on the bf16 matrix instructions: the three-term splitting of Henry, Tang and Heinecke, "Leveraging the
// bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations" (2019).
//
// A finite fp32 value of magnitude 2^-110 or more is the exact sum of three bf16 values: a high one (the nearest, or the one
// towards zero), the nearest to the remainder (middle) and what is left (low).  Below 2^-110 the low value falls under the
// smallest bf16 and the sum is off by up to 2^-133.  The product of two split values has nine partial products, each exact in fp32;
// the matrix instruction accumulates in fp32.  Six are kept where the multiplies are the bound,
//   low * high + high * low + middle * middle + middle * high + high * middle + high * high,
// and low * middle + middle * low as well where they are not.  With nearest high values |middle| <= 2^-8 and |low| <= 2^-17
// of the value's power of two, so six leave out at most 2^-24 of the product of the two powers of two; with one operand's
// towards zero (twice as large a middle and low value) 2^-23, with both 2^-22; eight always less than 2^-31.
//
// Error against 64 bits relative to the sum of the terms' magnitudes, root mean square / largest of a million sums of normally
// distributed products (emulated, small and large partial products summed apart):
//   terms               1                 2                 4                 16
//   fp32 multiply-adds  2.5e-8 / 5.9e-8   2.6e-8 / 1.2e-7   2.7e-8 / 1.7e-7   2.8e-8 / 2.5e-7
//   six, both nearest   2.6e-8 / 9.8e-8   2.2e-8 / 9.0e-8   1.7e-8 / 7.8e-8   1.0e-8 / 5.9e-8      convolutions
//   eight, towards zero 2.5e-8 / 6.0e-8   2.1e-8 / 6.0e-8   1.7e-8 / 6.0e-8   0.9e-8 / 5.7e-8      dense layers' gradients
//   six, towards zero   3.4e-8 / 2.4e-7   2.9e-8 / 2.2e-7   2.3e-8 / 1.8e-7   1.3e-8 / 9.1e-8      (not used)
// Rows of the dense average (weights nearest, parameters towards zero, six; measured): 2.2e-8, 2.0e-8 and 1.4e-8 for 2, 3 and 5
// terms, the fp32 instruction 2.2e-8, 2.4e-8 and 2.4e-8; its rows of one term have the weight 1, which splits into itself.
//
// v_mfma_f32_32x32x16_bf16 multiplies 16 times as many values per cycle as v_mfma_f32_32x32x2_f32 does, so six per 16-wide step
// have 2.7 times the rate: a register-resident loop reaches 312 TFLOP/s of fp32 products against 155 (212 to 246 when both
// operands are split in the loop as well).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace split_bf16 {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
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

// both rounded to bf16, a in the low 16 bits of the result
__device__ __forceinline__ uint32_t nearest(float a, float b)
{
    const bf16x2 r = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, r);
}

// The upper 16 bits of v as the high value: the nearest bf16, or, where that is infinite but v is not, the one towards zero.
__device__ __forceinline__ float high_value(float v)
{
    const uint32_t u = bits(v);
    return value((u & 0x7fffffffu) - 0x7f7f8000u < 0x8000u ? u & 0xffff0000u : nearest(v, v) << 16);
}

// Middle and low values of a and b, of which the high values h have been taken.
__device__ __forceinline__ void split_rest(float a, float b, uint32_t &m, uint32_t &l)
{
    m = nearest(a, b);
    a -= value(m << 16);
    b -= value(m & 0xffff0000u);
    l = upper(a, b);
}

// Eight values with the high value towards zero (the upper 16 bits): 11 vector instructions for two values.  The high value of a
// finite one is finite, an infinity is one in the high plane and NaN in the others; so is a NaN that has no bit among the upper 16
// bits' fraction (no instruction makes one).
__device__ __forceinline__ planes split8(const float (&x)[8])
{
    planes p;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float a = x[2 * q], b = x[2 * q + 1];
        uint32_t m, l;
        p.h[q] = upper(a, b);
        split_rest(a - value(bits(a) & 0xffff0000u), b - value(bits(b) & 0xffff0000u), m, l);
        p.m[q] = m;
        p.l[q] = l;
    }
    return p;
}

// N values (an even number) with the nearest high value, as pairs: 12 instructions for two.  An infinity or a NaN is one in the high
// plane and NaN in the others.  The half step below the largest float rounds to an infinite bf16, which shows as an infinite remainder
// (that of an infinity is NaN, which the maximum passes over): then once more, with high values that stay finite.
template <int N>
__device__ __forceinline__ void split_nearest(const float (&x)[N], uint32_t (&h)[N / 2], uint32_t (&m)[N / 2], uint32_t (&l)[N / 2])
{
    float rest = 0.f;
#pragma unroll
    for (int q = 0; q < N / 2; ++q) {
        h[q] = nearest(x[2 * q], x[2 * q + 1]);
        const float a = x[2 * q] - value(h[q] << 16), b = x[2 * q + 1] - value(h[q] & 0xffff0000u);
        rest = fmaxf(rest, fmaxf(fabsf(a), fabsf(b)));
        split_rest(a, b, m[q], l[q]);
    }
    if (__builtin_expect(rest == __builtin_inff(), 0)) {
#pragma unroll
        for (int q = 0; q < N / 2; ++q) {
            const float ha = high_value(x[2 * q]), hb = high_value(x[2 * q + 1]);
            split_rest(x[2 * q] - ha, x[2 * q + 1] - hb, m[q], l[q]);
            h[q] = upper(ha, hb);
        }
    }
}
// Eight of them into planes: written out, because as a call of split_nearest the compiler schedules the dense average otherwise, up to 6 %
// slower (36 workers x 3 M columns, local step first, a rate per worker: 385 -> 408 us).
__device__ __forceinline__ planes split8_nearest(const float (&x)[8])
{
    planes p;
    float rest = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t m, l;
        const uint32_t h = nearest(x[2 * q], x[2 * q + 1]);
        const float a = x[2 * q] - value(h << 16), b = x[2 * q + 1] - value(h & 0xffff0000u);
        rest = fmaxf(rest, fmaxf(fabsf(a), fabsf(b)));
        split_rest(a, b, m, l);
        p.h[q] = h;
        p.m[q] = m;
        p.l[q] = l;
    }
    if (__builtin_expect(rest == __builtin_inff(), 0)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float ha = high_value(x[2 * q]), hb = high_value(x[2 * q + 1]);
            uint32_t m, l;
            split_rest(x[2 * q] - ha, x[2 * q + 1] - hb, m, l);
            p.h[q] = upper(ha, hb);
            p.m[q] = m;
            p.l[q] = l;
        }
    }
    return p;
}

__device__ __forceinline__ bf16x8 frag(const u32x4 &v) { return __builtin_bit_cast(bf16x8, v); }

// large + small += a b over 16 terms (32 x 32 outputs).  Lane l holds row (or column) l % 32 of the operand and the terms 8 (l / 32) ..
// + 7 of the step: any assignment of terms to lanes that is the same for both operands gives the same sums.  The large partial
// products, of 16 bits each, have an accumulator of their own, which is rounded once per 16 terms and for a few terms hardly at all;
// the sum of the two (the caller's) is two to three times closer to the exact one than a single accumulator (9e-8 at
// 256 terms, 1.6e-7 at 800); also two shorter chains of dependent instructions.  ALL: eight partial products.
template <bool ALL>
__device__ __forceinline__ void mma32(const planes &a, const planes &b, f32x16 &large, f32x16 &small)
{
    if (ALL) {
        small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.l), frag(b.m), small, 0, 0, 0);
        small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.m), frag(b.l), small, 0, 0, 0);
    }
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.l), frag(b.h), small, 0, 0, 0);
    large = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.h), frag(b.h), large, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.h), frag(b.l), small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.m), frag(b.m), small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.m), frag(b.h), small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a.h), frag(b.m), small, 0, 0, 0);
}

// one matrix instruction: 32 x 32 outputs over 16 terms, or 16 x 16 over 32 (lane l: row or column l % 16, terms 8 (l / 16) .. + 7)
__device__ __forceinline__ void mma(const u32x4 &a, const u32x4 &b, f32x16 &acc)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(a), frag(b), acc, 0, 0, 0);
}
__device__ __forceinline__ void mma(const u32x4 &a, const u32x4 &b, f32x4 &acc)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(a), frag(b), acc, 0, 0, 0);
}

// One sparse matrix instruction: 32 x 32 outputs over 32 terms, of which every four in a row have at most two nonzero values of a, in the
// time of mma's 16.  Lane l of b holds column l % 32 and the terms 16 (l / 32) .. + 15.  Lane l of a holds row l % 32 and, in pairs, the values
// of the terms 8 (l / 32) + 0 .. 3, + 4 .. 7, 16 + 8 (l / 32) + 0 .. 3 and + 4 .. 7; four bits of `index` for each pair, from bit 0 on, say
// which two of its four terms they are, the first one's place in the lower two bits (layout as probed on the card: every place of
// every pair, against b = the terms' numbers).
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ void mma_sparse(const u32x4 &a, const u32x8 &b, int index, f32x16 &acc)
{
    acc = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(frag(a), __builtin_bit_cast(bf16x16, b), acc, index, 0, 0);
}

// Six partial products (or the five small ones, or the large one) for a block of A x B accumulators, one kind after the other,
// the large one last: consecutive instructions are independent.
template <bool SMALL, bool LARGE, int A, int B, class Acc>
__device__ __forceinline__ void mma_block(const planes (&a)[A], const planes (&b)[B], Acc (&acc)[A][B])
{
    auto step = [&](u32x4 planes::*pa, u32x4 planes::*pb) {
#pragma unroll
        for (int i = 0; i < A; ++i)
#pragma unroll
            for (int j = 0; j < B; ++j) mma(a[i].*pa, b[j].*pb, acc[i][j]);
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
template <class Acc>
__device__ __forceinline__ bool any_not_finite(const Acc &acc)
{
    float t = 0.f;
#pragma unroll
    for (int v = 0; v < (int)(sizeof(Acc) / 4); ++v) t = fmaf(acc[v], 0.f, t);
    return t != t;
}

// large += small, where large is finite.  The high plane holds an infinity or NaN as what it is and zero as zero, so a large sum
// that is not finite is what fp32 multiply-adds give (a factor below 2^-133 counts as zero next to an infinity); the small one is
// then NaN for reasons of its own (a middle value next to an infinity has either sign or is zero).
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
template <class Acc>
__device__ __forceinline__ void drop_not_finite(Acc &small)
{
#pragma unroll
    for (int v = 0; v < (int)(sizeof(Acc) / 4); ++v) small[v] = not_finite(small[v]) ? 0.f : small[v];
}

}  // namespace split_bf16
