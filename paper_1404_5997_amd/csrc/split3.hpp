// fp32 products on the bf16 matrix unit: every fp32 operand is written as the sum of three bf16 values,
//     v = h + m + l,   h = bf16(v),  m = bf16(v - h),  l = bf16(v - h - m),
// which is exact (3 x 8 significant bits) where none of the parts leaves bf16's range, and of the nine products of two such
// sums the six largest are taken:
//     v*w ~ h*h' + (h*m' + m*h') + (m*m' + h*l' + l*h'),
// leaving out m*l' + l*m' + l*l', at most 2^-24 |v*w| together (|m| <= 2^-8 |v|, |l| <= 2^-17 |v|).  A bf16 product is exact in
// fp32, so what is left is the rounding of the accumulators.  h*h' is added up in one accumulator and the five small products in
// another; the two are added once at the end.  Each 16-deep matrix instruction rounds its accumulator once, so a reduction of length L rounds the large
// accumulator L/16 times where the fp32 matrix instruction (2 deep) rounds L/2 times.  Measured against 64 bits on
// sums of normally distributed products, relative 2-norm error, fp32 instruction -> this scheme: length 576
// 4.3e-7 -> 1.4e-7, 1728 7.4e-7 -> 2.5e-7, 4800 1.2e-6 -> 4.3e-7, 23328 2.7e-6 -> 9.8e-7.  (All six products in one
// accumulator: 6.4e-7 at 1728, and 1.0e-6 where the fp32 instruction has 8.7e-7 at 4800 when one operand is >= 0: not
// used.)  The bf16 matrix rate is 16 times the fp32 one, so six products cost 6/16 of an fp32 instruction's time.
//
// The ends of the range.  Below 2^-110 the small parts fall out of bf16's range and an operand loses bits; within 2^-8 of the
// largest number h*h' can be infinite where v*w is not.  So either the operands are scaled by 2^24 each as they are split (the
// smallest subnormal number then has all its parts; one multiplication a value), the result by 2^-48, and what leaves the
// range at the top (a value past 2^104, a sum past 2^80) is worked out again unscaled; or, where that multiplication would be felt, the
// plain split comes first and a result that shows either end is worked out again, scaled up or down.
#pragma once
#include "owt_common.hpp"

namespace owt {

typedef __bf16 split_frag __attribute__((ext_vector_type(8)));         // one operand fragment of the 32x32x16 instruction
typedef float split_acc __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float bf16_lo_f32(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf16_hi_f32(uint32_t pair) { return __uint_as_float(pair & 0xffff0000u); }
__device__ __forceinline__ float sum8_bf16(uint4 q)
{
    return ((bf16_lo_f32(q.x) + bf16_hi_f32(q.x)) + (bf16_lo_f32(q.y) + bf16_hi_f32(q.y))) +
           ((bf16_lo_f32(q.z) + bf16_hi_f32(q.z)) + (bf16_lo_f32(q.w) + bf16_hi_f32(q.w)));
}

constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;
// A result below this, and not zero, is worked out again scaled.  A larger one has lost less than 2^-24 of it to operands below
// 2^-110 as long as the values these were multiplied with add up to less than 2^46.  (A result of zero stays: the plain split takes
// operands below 2^-134 for zero.  And a tile that holds such a result beside one past 2^80 keeps what the second scale gives.)
constexpr float kSplitTiny = 0x1p-64f;
// Scales of the two operands for the second run of a result that was not finite: no product leaves the range that fits in it.
constexpr float kSplitDown = 0x1p-2f, kSplitUndown = 4.f;

// Values the plain rule cannot split: h would round to infinity (|v| >= 0x1.ffp127, finite) or v is infinite.
// Finite: h = v truncated to bf16, the rest as above.  Infinite: h = +-1, m = 0, l = v, so that every product with a
// non-zero finite value is that infinity (once, from l*h') and nothing else is infinite.  NaN takes the plain rule.
__device__ __forceinline__ void split3_one_large(float v, uint16_t &h, uint16_t &m, uint16_t &l)
{
    const uint32_t b = __float_as_uint(v);
    if ((b & 0x7fffffffu) == 0x7f800000u) {
        h = (uint16_t)((b >> 16 & 0x8000u) | 0x3f80u);
        m = 0;
        l = (uint16_t)(b >> 16);
        return;
    }
    float hf = __uint_as_float(f32x2_to_bf16x2(v, 0.f) << 16);
    if ((__float_as_uint(hf) & 0x7fffffffu) == 0x7f800000u) hf = __uint_as_float(b & 0xffff0000u);
    const float r = v - hf;
    const uint32_t mb = f32x2_to_bf16x2(r, 0.f) & 0xffffu;
    h = (uint16_t)(__float_as_uint(hf) >> 16);
    m = (uint16_t)mb;
    l = (uint16_t)(f32x2_to_bf16x2(r - __uint_as_float(mb << 16), 0.f) & 0xffffu);
}

// Eight values into three fragments: 5.5 vector instructions per value and half a one for the test of the rare case.
__device__ __forceinline__ void split3_careful(const float (&v)[8], split_frag (&f)[3])
{
    uint32_t hh[4], mm[4], ll[4];
    float top = 0.f;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const float a = v[2 * i], b = v[2 * i + 1];
        asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(top) : "v"(a), "v"(b));       // fmaxf() adds a canonicalisation per value
        hh[i] = f32x2_to_bf16x2(a, b);
        const float ra = a - bf16_lo_f32(hh[i]), rb = b - bf16_hi_f32(hh[i]);
        mm[i] = f32x2_to_bf16x2(ra, rb);
        ll[i] = f32x2_to_bf16x2(ra - bf16_lo_f32(mm[i]), rb - bf16_hi_f32(mm[i]));
    }
    if (top >= 3.38e38f) {                       // some |v| near or past the largest bf16 (NaN does not count)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            uint16_t h0, m0, l0, h1, m1, l1;
            split3_one_large(v[2 * i], h0, m0, l0);
            split3_one_large(v[2 * i + 1], h1, m1, l1);
            hh[i] = h0 | (uint32_t)h1 << 16; mm[i] = m0 | (uint32_t)m1 << 16; ll[i] = l0 | (uint32_t)l1 << 16;
        }
    }
    f[0] = __builtin_bit_cast(split_frag, make_uint4(hh[0], hh[1], hh[2], hh[3]));
    f[1] = __builtin_bit_cast(split_frag, make_uint4(mm[0], mm[1], mm[2], mm[3]));
    f[2] = __builtin_bit_cast(split_frag, make_uint4(ll[0], ll[1], ll[2], ll[3]));
}

// The same with no test: infinite values, and finite ones above the largest bf16, turn into NaN.
__device__ __forceinline__ void split3_plain(const float (&v)[8], split_frag (&f)[3])
{
    uint32_t hh[4], mm[4], ll[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        hh[i] = f32x2_to_bf16x2(v[2 * i], v[2 * i + 1]);
        const float ra = v[2 * i] - bf16_lo_f32(hh[i]), rb = v[2 * i + 1] - bf16_hi_f32(hh[i]);
        mm[i] = f32x2_to_bf16x2(ra, rb);
        ll[i] = f32x2_to_bf16x2(ra - bf16_lo_f32(mm[i]), rb - bf16_hi_f32(mm[i]));
    }
    f[0] = __builtin_bit_cast(split_frag, make_uint4(hh[0], hh[1], hh[2], hh[3]));
    f[1] = __builtin_bit_cast(split_frag, make_uint4(mm[0], mm[1], mm[2], mm[3]));
    f[2] = __builtin_bit_cast(split_frag, make_uint4(ll[0], ll[1], ll[2], ll[3]));
}

// Eight values scaled by kSplitScale into three pieces of packed bf16 (16 bytes each).  Infinite or NaN: h = 1 with the value's
// sign, m = 0, l = v, so that the sum of the small products becomes what fp32 products give and h*h' stays finite.  Finite and too
// large for the scale: h is infinite, and the sum of h*h' shows it.
__device__ __forceinline__ void split3_scaled(const float (&v)[8], uint4 &h, uint4 &m, uint4 &l)
{
    uint32_t hh[4], mm[4], ll[4];
    float top = 0.f;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const float a = v[2 * i] * kSplitScale, b = v[2 * i + 1] * kSplitScale;
        asm("v_maximum3_f32 %0, |%1|, |%2|, %0" : "+v"(top) : "v"(a), "v"(b));   // NaN if one is
        hh[i] = f32x2_to_bf16x2(a, b);
        const float ra = a - bf16_lo_f32(hh[i]), rb = b - bf16_hi_f32(hh[i]);
        mm[i] = f32x2_to_bf16x2(ra, rb);
        ll[i] = f32x2_to_bf16x2(ra - bf16_lo_f32(mm[i]), rb - bf16_hi_f32(mm[i]));
    }
    if (!(top < __builtin_inff())) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t odd = (fabsf(v[2 * i]) < __builtin_inff() ? 0u : 0xffffu) | (fabsf(v[2 * i + 1]) < __builtin_inff() ? 0u : 0xffff0000u);
            const uint32_t raw = f32x2_to_bf16x2(v[2 * i], v[2 * i + 1]);
            hh[i] = (hh[i] & ~odd) | (((raw & 0x80008000u) | 0x3f803f80u) & odd);
            mm[i] &= ~odd;
            ll[i] = (ll[i] & ~odd) | (raw & odd);
        }
    }
    h = make_uint4(hh[0], hh[1], hh[2], hh[3]);
    m = make_uint4(mm[0], mm[1], mm[2], mm[3]);
    l = make_uint4(ll[0], ll[1], ll[2], ll[3]);
}

}  // namespace owt
