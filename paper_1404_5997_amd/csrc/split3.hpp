// fp32 products on the bf16 matrix unit: every fp32 operand is written as the sum of three bf16 values,
//     v = h + m + l,   h = bf16(v),  m = bf16(v - h),  l = bf16(v - h - m),
// which is exact (3 x 8 significant bits) as long as l does not underflow (|v| below about 2^-110), and of the
// nine products of two such sums the six largest are taken:
//     v*w ~ h*h' + (h*m' + m*h') + (m*m' + h*l' + l*h'),
// leaving out terms of at most 2^-25 |v*w|.  A bf16 product is exact in fp32, so what is left is the rounding of the
// accumulators.  h*h' is added up in one accumulator and the five small products in another; the two are added once
// at the end.  Each 16-deep matrix instruction rounds its accumulator once, so a reduction of length L rounds the large
// accumulator L/16 times where the fp32 matrix instruction (2 deep) rounds L/2 times.  Measured against 64 bits on
// sums of normally distributed products, relative 2-norm error, fp32 instruction -> this scheme: length 576
// 4.3e-7 -> 1.4e-7, 1728 7.4e-7 -> 2.5e-7, 4800 1.2e-6 -> 4.3e-7, 23328 2.7e-6 -> 9.8e-7.  (All six products in one
// accumulator: 6.4e-7 at 1728, and 1.0e-6 where the fp32 instruction has 8.7e-7 at 4800 when one operand is >= 0: not
// used.)  The bf16 matrix rate is 16 times the fp32 one, so six products cost 6/16 of an fp32 instruction's time.
#pragma once
#include "owt_common.hpp"

namespace owt {

typedef __bf16 split_frag __attribute__((ext_vector_type(8)));         // one operand fragment of the 32x32x16 instruction
typedef float split_acc __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float bf16_lo_f32(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf16_hi_f32(uint32_t pair) { return __uint_as_float(pair & 0xffff0000u); }

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

// Eight values into three fragments' worth of packed bf16 (16 bytes each): 5.5 vector instructions per value and
// half a one for the test of the rare case.
__device__ __forceinline__ void split3_pack8(const float (&v)[8], uint4 &h, uint4 &m, uint4 &l)
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
    h = make_uint4(hh[0], hh[1], hh[2], hh[3]);
    m = make_uint4(mm[0], mm[1], mm[2], mm[3]);
    l = make_uint4(ll[0], ll[1], ll[2], ll[3]);
}

// The six products of one fragment pair; a[0..2], b[0..2] = h, m, l.  Small products first, their own accumulator.
__device__ __forceinline__ void split3_small(const split_frag (&a)[3], const split_frag (&b)[3], split_acc &small)
{
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], small, 0, 0, 0);
}

}  // namespace owt
