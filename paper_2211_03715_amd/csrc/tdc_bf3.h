// fp32 products on the bf16 matrix cores, shared by the kernels that are bound by matrix arithmetic.
//
// gfx950 multiplies fp32 at 157 TFLOP/s and bf16 at 2500.  A finite fp32 value is the sum of three bf16 values,
//     v = v1 + v2 + v3,   v1 = bf16(v), v2 = bf16(v - v1), v3 = v - v1 - v2   (24 = 3 x 8 significand bits; the
//     subtractions are exact), |v2| <= 2^-8 |v|, |v3| <= 2^-16 |v|,
// so a product a*b is nine exact bf16 products.  Six of them are accumulated (in fp32, by the matrix core):
//     a3 b1 + a2 b2 + a1 b3 + a2 b1 + a1 b2 + a1 b1;
// the three left out are together below 2^-23 |a b| in the worst case and about 2^-26 |a b| on average.  A chain of n
// fp32 multiply-adds, which this replaces, may be off by n * 2^-24 sum |a b|; the split product by 2 * 2^-24 sum |a b|
// plus the roundings of n/32 accumulations, so from n = 3 on its bound is the smaller one (the selector leaves shorter sums to
// the fp32 kernels).  Measured against fp64 on
// normal inputs (one 16 x 16 block): relative error 3.7e-8 / 2.3e-7 / 5.7e-7 / 1.1e-6 at n = 32 / 256 / 1152 / 4608, where
// v_mfma_f32_16x16x4_f32 gives 1.1e-7 / 3.1e-7 / 7.1e-7 / 1.3e-6; all nine products give the same figures as six.
// Time per 16 x 16 x 32 block: 6 x 16 cycles against 8 x 32.
// Values below 2^-110 keep an absolute accuracy of 2^-134 instead of a relative one (bf16 has no smaller subnormals).  Beside
// larger ones that is below their rounding; a sum of which nothing is larger would lose bits.
// Infinities have no three parts, nor have finite values the conversion rounds to infinity (above 3.39e38): split, they give
// NaN (inf - inf).  Where parts are stored such a value, like every one from 2^126 on, is kept raw: its fp32 bits in the
// second and third part, behind a first part that is a NaN (TDC_RAW).  Either way every sum it reaches is NaN; a kernel that
// ends up with a NaN or a magnitude from 2^126 on computes those sums once more with fp32 multiply-adds on the joined parts.
// The same where all sums of a pixel that a lane or wavefront holds are below 2^-76 and not zero, as they are if no factor
// there reaches 2^-110: weights of a tensor whose largest is outside 2^-100 .. 2^14 are kept raw, every one, so that a tensor
// in parts cannot lift such a factor above that (2^20 terms of 2^14 * 2^-110).
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

__device__ __forceinline__ tdc_u2 tdc_buf_load2(tdc_rsrc r, unsigned byte_off)
{
    return __builtin_bit_cast(tdc_u2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)byte_off, 0, 0));
}

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

// Largest magnitude, NaN if one is (v_maximum3_f32: two values an instruction).
constexpr float TDC_BIG = 0x1p126f, TDC_SMALL = 0x1p-76f;
__device__ __forceinline__ float tdc_largest(float m, tdc_f4 v)
{
    m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, fabsf(v[0])), fabsf(v[1]));
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, fabsf(v[2])), fabsf(v[3]));
}
// The smallest of several magnitudes that is not zero, as an integer: start with ~0u.
__device__ __forceinline__ unsigned tdc_smallest(unsigned s, float m) { return min(s, __builtin_bit_cast(unsigned, m) - 1u); }
constexpr unsigned TDC_SMALL_BITS = (127u - 76u) << 23;
__device__ __forceinline__ bool tdc_is_small(unsigned s) { return s < TDC_SMALL_BITS - 1u; }
__device__ __forceinline__ bool tdc_any_lane(bool b) { return __builtin_amdgcn_ballot_w64(b) != 0; }

// first part of a value whose fp32 bits are the other two
constexpr unsigned TDC_RAW = 0x7fffu;

// tdc_split2 for values that are stored: those from 2^126 on or not zero and below `least` are kept raw (a NaN is a NaN in
// every part)
__device__ __forceinline__ void tdc_split2_raw(float a, float b, float least, unsigned &p1, unsigned &p2, unsigned &p3)
{
    tdc_split2(a, b, p1, p2, p3);
    const unsigned ua = __builtin_bit_cast(unsigned, a), ub = __builtin_bit_cast(unsigned, b);
    if (!(fabsf(a) < TDC_BIG) || (a != 0.f && fabsf(a) < least)) {
        p1 = (p1 & 0xffff0000u) | (a != a ? 0x7fc0u : TDC_RAW);
        p2 = (p2 & 0xffff0000u) | ua >> 16;
        p3 = (p3 & 0xffff0000u) | (ua & 0xffffu);
    }
    if (!(fabsf(b) < TDC_BIG) || (b != 0.f && fabsf(b) < least)) {
        p1 = (p1 & 0xffffu) | (b != b ? 0x7fc0u : TDC_RAW) << 16;
        p2 = (p2 & 0xffffu) | (ub & 0xffff0000u);
        p3 = (p3 & 0xffffu) | ub << 16;
    }
}

// the fp32 value of stored parts
__device__ __forceinline__ float tdc_join(unsigned p1, unsigned p2, unsigned p3)
{
    const auto part = [](unsigned v) { return __builtin_bit_cast(float, v << 16); };
    return p1 == TDC_RAW ? __builtin_bit_cast(float, p2 << 16 | p3) : part(p1) + (part(p2) + part(p3));
}
__device__ __forceinline__ tdc_f4 tdc_join4(const tdc_u2 (&p)[3])
{
    tdc_f4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const unsigned u[3] = {p[0][j >> 1], p[1][j >> 1], p[2][j >> 1]};
        v[j] = j & 1 ? tdc_join(u[0] >> 16, u[1] >> 16, u[2] >> 16) : tdc_join(u[0] & 0xffffu, u[1] & 0xffffu, u[2] & 0xffffu);
    }
    return v;
}

// k-group kg's share of a lane's weights of 16-channel block `block`, from the three-part layout (tdc_internal.h)
__device__ __forceinline__ tdc_f4 tdc_join_weights(tdc_rsrc r, int block, int steps, int kg, int lane)
{
    tdc_u2 p[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) p[q] = tdc_buf_load2(r, (unsigned)(block * steps + (kg >> 1)) * 3072u + q * 1024u + lane * 16u + 8u * (kg & 1));
    return tdc_join4(p);
}
__device__ __forceinline__ tdc_u2 tdc_first_parts(tdc_rsrc r, int block, int steps, int kg, int lane)
{
    return tdc_buf_load2(r, (unsigned)(block * steps + (kg >> 1)) * 3072u + lane * 16u + 8u * (kg & 1));
}

// Whether the NaNs among some sums can only come from NaNs among their factors: there is one, and the other factors are too
// small for products or sums of three stages to overflow.
struct TdcFactors {
    float largest = 0.f;       // magnitude of the largest that is not NaN
    bool nan = false, low = false;     // low: one below 2^-38 that is not 0; without, no product of two is small (2^-76)
    __device__ __forceinline__ void see(tdc_f4 v)
    {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            nan |= v[j] != v[j];
            largest = fmaxf(largest, fabsf(v[j]));
            low |= v[j] != 0.f && fabsf(v[j]) < 0x1p-38f;
        }
    }
    // four stored values by their first parts
    __device__ __forceinline__ void see(tdc_u2 p1)
    {
        tdc_f4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const unsigned u = p1[j >> 1] >> 16 * (j & 1) & 0xffffu;
            v[j] = __builtin_bit_cast(float, u == TDC_RAW ? 0x7f800000u : u << 16);
        }
        see(v);
    }
    __device__ __forceinline__ bool explain_nan() const { return tdc_any_lane(nan) && !tdc_any_lane(largest >= 0x1p30f); }
};

// The kernel's arguments (its one parameter), read anew where this is called: what is hardly ever run keeps no registers of what
// always is.
template <class Args>
__device__ __forceinline__ const Args &tdc_args_again()
{
    typedef const __attribute__((address_space(4))) Args *Ptr;
    Ptr p = (Ptr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const Args *)p;
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

__device__ __forceinline__ void tdc_split4_raw(tdc_f4 v, float least, tdc_u2 &p1, tdc_u2 &p2, tdc_u2 &p3)
{
    unsigned a1, a2, a3, b1, b2, b3;
    tdc_split2_raw(v[0], v[1], least, a1, a2, a3);
    tdc_split2_raw(v[2], v[3], least, b1, b2, b3);
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

#endif
