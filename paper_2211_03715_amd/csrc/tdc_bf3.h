// fp32 products on the bf16 matrix cores, shared by the kernels that are bound by matrix arithmetic.
//
// gfx950 multiplies fp32 at 157 TFLOP/s and bf16 at 2500.  A finite fp32 value is the sum of three bf16 values,
//     v = v1 + v2 + v3,   v1 = bf16(v), v2 = bf16(v - v1), v3 = v - v1 - v2   (24 = 3 x 8 significand bits; the
//     subtractions are exact), |v2| <= 2^-8 |v|, |v3| <= 2^-16 |v|,
// so a product a*b is nine exact bf16 products.  Six of them are accumulated (in fp32, by the matrix core):
//     a3 b1 + a2 b2 + a1 b3 + a2 b1 + a1 b2 + a1 b1;
// the three left out are together below 2^-23 |a b| in the worst case and about 2^-26 |a b| on average.  A chain of n
// fp32 multiply-adds, which this replaces, may be off by n * 2^-24 sum |a b|; the split product by 2 * 2^-24 sum |a b|
// plus the roundings of n/32 accumulations, so from n = 3 on its bound is the smaller one.  Measured against fp64 on
// normal inputs (one 16 x 16 block): relative error 3.7e-8 / 2.3e-7 / 5.7e-7 / 1.1e-6 at n = 32 / 256 / 1152 / 4608, where
// v_mfma_f32_16x16x4_f32 gives 1.1e-7 / 3.1e-7 / 7.1e-7 / 1.3e-6; all nine products give the same figures as six.
// Time per 16 x 16 x 32 block: 6 x 16 cycles against 8 x 32.
// Values below 2^-110 keep an absolute accuracy of 2^-134 instead of a relative one (bf16 has no smaller subnormals);
// an infinite value comes out as NaN (inf - inf in the split): a kernel whose fp32 form gave infinities looks for that.
//
// Operand layout of v_mfma_f32_16x16x32_bf16 (D 16x16 += A 16x32 * B 32x16): lane l holds A[m = l%16][k(l/16, j)] and
// B[k(l/16, j)][p = l%16], j = 0..7, for any assignment k(g, j) that A and B share; D as in tdc_mfma.h.  Here a step is a pair of
// 16-wide k-groups of the enumeration every kernel of this library uses, and k(g, j) = component j%4 of lane group g in
// group j/4 of the pair: channel 4g + j%4.  As there, the four accumulator registers of a lane after one stage are its
// operand half in the next.
#ifndef TDC_BF3_H
#define TDC_BF3_H

#include "tdc_mfma.h"

typedef __bf16 tdc_bf8 __attribute__((ext_vector_type(8)));
typedef unsigned tdc_u2 __attribute__((ext_vector_type(2)));
typedef unsigned tdc_u4 __attribute__((ext_vector_type(4)));

// two fp32 -> their three bf16 parts, packed in pairs (11 VALU instructions)
__device__ __forceinline__ void tdc_split2(float a, float b, unsigned &p1, unsigned &p2, unsigned &p3)
{
    // Opaque after the conversion: the compiler would else convert the low value a second time rather than shift the pair.
    // The conversion itself must not be written as asm: it may read a matrix-core result, and the compiler inserts the wait
    // states that needs only in front of instructions it knows.
    const auto pack = [](float u, float v) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
        unsigned r = __builtin_bit_cast(unsigned, __builtin_convertvector((f2){u, v}, bf2));
        asm("" : "+v"(r));
        return r;
    };
    p1 = pack(a, b);
    const float ra = a - __builtin_bit_cast(float, p1 << 16), rb = b - __builtin_bit_cast(float, p1 & 0xffff0000u);
    p2 = pack(ra, rb);
    p3 = pack(ra - __builtin_bit_cast(float, p2 << 16), rb - __builtin_bit_cast(float, p2 & 0xffff0000u));
}

// four fp32 (one lane's share of a 16-wide k-group) -> three 8-byte operand halves
__device__ __forceinline__ void tdc_split4(tdc_f4 v, tdc_u2 &p1, tdc_u2 &p2, tdc_u2 &p3)
{
    unsigned a1, a2, a3, b1, b2, b3;
    tdc_split2(v[0], v[1], a1, a2, a3);
    tdc_split2(v[2], v[3], b1, b2, b3);
    p1 = (tdc_u2){a1, b1};
    p2 = (tdc_u2){a2, b2};
    p3 = (tdc_u2){a3, b3};
}

// one operand of a 32-wide step in its three parts
struct tdc_op3 {
    tdc_bf8 p[3];
};

// a lane's operand from its shares of the two k-groups of a step
__device__ __forceinline__ tdc_op3 tdc_split_op(tdc_f4 lo, tdc_f4 hi)
{
    tdc_u2 a[3], b[3];
    tdc_split4(lo, a[0], a[1], a[2]);
    tdc_split4(hi, b[0], b[1], b[2]);
    tdc_op3 o;
#pragma unroll
    for (int i = 0; i < 3; ++i) o.p[i] = __builtin_bit_cast(tdc_bf8, (tdc_u4){a[i][0], a[i][1], b[i][0], b[i][1]});
    return o;
}

__device__ __forceinline__ tdc_f4 tdc_mfma_bf(tdc_bf8 a, tdc_bf8 b, tdc_f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The six products, smallest first: parts of A and of B.
constexpr int TDC_BF3_A[6] = {2, 1, 0, 1, 0, 0}, TDC_BF3_B[6] = {0, 1, 2, 0, 1, 0};

// acc[mb][pb] += A(mb) * B(pb) over one 32-wide step.  SWAP: B supplies the rows of D (pixels) and A its columns.
template <int MB, int PB, bool SWAP = false>
__device__ __forceinline__ void tdc_mma3(tdc_f4 (&acc)[MB][PB], const tdc_op3 (&a)[MB], const tdc_op3 (&b)[PB])
{
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
                acc[mb][pb] = SWAP ? tdc_mfma_bf(b[pb].p[TDC_BF3_B[i]], a[mb].p[TDC_BF3_A[i]], acc[mb][pb])
                                   : tdc_mfma_bf(a[mb].p[TDC_BF3_A[i]], b[pb].p[TDC_BF3_B[i]], acc[mb][pb]);
}

#endif
