// fp32 products on the fp16 matrix cores, shared by the kernels that are bound by matrix arithmetic.
//
// gfx950 multiplies fp32 at 157 TFLOP/s and fp16 at 2500.  A value that has been scaled by a power of two into fp16's range is
//     v = v1 + 2^-11 (v2 + v3),   v1 = fp16(v), v2 = fp16(2^11 (v - v1)), v3 = fp16(2^11 (v - v1) - v2):
// the parts have 11 significand bits each, so two of them are off by at most half a bit of the 24 (v3 is what is left).
// The products of parts i and j with i + j < parts are accumulated, in fp32 by the matrix core, in two accumulators ("levels"), the
// second of which is 2^11 times the sum and is added at the end.  Three parts of a weight are not lifted, w = w1 + w2 + w3, so
// that their products need no third one:
//     two parts:    w1 x1 | w1 x2 + w2 x1                                      3 MFMAs of 16 cycles per 16 x 16 x 32 block
//     three parts:  w1 x1 + w2 x1 + w3 x1 | w1 x2 + w2 x2 + w1 x3              6 (fp32 MFMA: 8 of 32)
// Only the accumulations of the highest level round at the scale of the result, n/32 of them.  Measured against 64 bits
// (normal values, relative 2-norm): at n = 32 / 64 / 128 / 288 / 1152 / 4608 terms two parts 9.0e-8 / 9.7e-8 / 1.1e-7 / 1.4e-7 /
// 2.3e-7 / 4.4e-7; three bf16 parts in one accumulator (tdc_bf3.h) 3.8e-8 / 9.3e-8 / 1.6e-7 / 2.4e-7 / 5.1e-7 / 1.08e-6;
// v_mfma_f32_16x16x4_f32 1.0e-7 / 1.4e-7 / 2.0e-7 / 3.1e-7 / 6.0e-7 / 1.2e-6.  Sums too short for two parts to be the most
// accurate of these take three or, in most kernels, three bf16 ones (tdc_tile_parts, tdc_chain3_bf3).
//
// Scales.  fp16 holds 2^-24 .. 65504, so v2 keeps its 11 bits down to |v| = 2^-13 and the parts an absolute 2^-36 below that.
//   weights      every output channel has its own exponent, the largest weight at 2^13 .. 2^14 (tdc_pack.hip): three parts that
//                are not lifted keep all 24 bits down to 2^-1 and an absolute 2^-25 below, 2^-38 of the largest weight;
//   activations  one exponent per workgroup, which takes the largest magnitude among those it loads first to 2^6 .. 2^7
//                (tdc_scale_of): 512 times larger values still fit, 2^19 times smaller ones keep all their bits (from 2^10 on
//                it would be 64 times and 2^23: channels of larger values behind the first ones are the commoner thing);
//   z1           sqrt(C) 2^11 times smaller than its sums, a constant: 2^5 or so, and below 2^14 where all signs agree;
//   z2           by the largest a wavefront holds.
// What is lost.  A factor below 2^TDC_LOWEST is kept to an absolute accuracy, 2^-36.  That shows where large weights meet small
// values only, as when the weights undo what size the channels of x have: the sums are small then, a channel's over several
// pixels (one or two may be so by chance), and each stage that writes outputs compares them with what the parts may have lost.
// Infinities, NaN and values too large show in the results, which they make infinite or NaN; that all of a pixel's channels are
// below 2^-13, and not zero, each stage watches as it splits them (a pixel's, not a value's: beside larger ones a lost bit is
// below their rounding, unless weights undo the difference, which is what the outputs are compared for).  Either way the outputs concerned are computed once more in fp32, from weights kept beside the parts.
//
// Operand layout of v_mfma_f32_16x16x32_f16 (D 16x16 += A 16x32 * B 32x16): lane l holds A[m = l%16][k(l/16, j)] and
// B[k(l/16, j)][p = l%16], j = 0..7, for any assignment k(g, j) that A and B share; D as in tdc_mfma.h.  Here a step is a pair of
// 16-wide k-groups of the enumeration every kernel of this library uses, and k(g, j) = component j%4 of lane group g in
// group j/4 of the pair: channel 4g + j%4.  As there, the four accumulator registers of a lane after one stage are its
// operand half in the next.
#ifndef TDC_SPLIT_H
#define TDC_SPLIT_H

#include "tdc_mfma.h"

typedef _Float16 tdc_h2 __attribute__((ext_vector_type(2)));
typedef _Float16 tdc_h8 __attribute__((ext_vector_type(8)));
typedef unsigned tdc_u2 __attribute__((ext_vector_type(2)));
typedef unsigned tdc_u4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ tdc_u2 tdc_buf_load2(tdc_rsrc r, unsigned byte_off)
{
    return __builtin_bit_cast(tdc_u2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)byte_off, 0, 0));
}

// 2^e, e in -126 .. 127
__device__ __forceinline__ float tdc_exp2i(int e) { return __builtin_bit_cast(float, (unsigned)(127 + e) << 23); }

// a power of two to scale by, and 2^11 times it
struct TdcScale {
    float one, lift;
    __device__ __forceinline__ explicit TdcScale(int e) : one(tdc_exp2i(e)), lift(tdc_exp2i(e + 11)) {}
};

// two scaled fp32 -> their parts, packed in pairs (two parts: 7 VALU instructions); LIFT: the parts behind the first times 2^11
template <int NP, bool LIFT = true>
__device__ __forceinline__ void tdc_split2(float a, float b, const TdcScale &s, unsigned (&p)[NP])
{
    // Opaque after the conversion: the compiler would else convert each value a second time for its rest.  The conversion itself
    // must not be written as asm: it may read a matrix-core result, and the compiler inserts the wait states that needs only in
    // front of instructions it knows.
    const auto pack = [](float u, float v) {
        unsigned r = __builtin_bit_cast(unsigned, (tdc_h2){(_Float16)u, (_Float16)v});
        asm("" : "+v"(r));
        return r;
    };
    p[0] = pack(a * s.one, b * s.one);
    float ra = a * (LIFT ? s.lift : s.one), rb = b * (LIFT ? s.lift : s.one);
#pragma unroll
    for (int q = 1; q < NP; ++q) {
        const tdc_h2 v = __builtin_bit_cast(tdc_h2, p[q - 1]);
        ra = fmaf((float)v[0], LIFT && q == 1 ? -2048.f : -1.f, ra);
        rb = fmaf((float)v[1], LIFT && q == 1 ? -2048.f : -1.f, rb);
        p[q] = q + 1 < NP ? pack(ra, rb) : __builtin_bit_cast(unsigned, (tdc_h2){(_Float16)ra, (_Float16)rb});
    }
}

// four fp32 (one lane's share of a 16-wide k-group) -> 8-byte operand halves
template <int NP>
__device__ __forceinline__ void tdc_split4(tdc_f4 v, const TdcScale &s, tdc_u2 (&p)[NP])
{
    unsigned a[NP], b[NP];
    tdc_split2<NP>(v[0], v[1], s, a);
    tdc_split2<NP>(v[2], v[3], s, b);
#pragma unroll
    for (int q = 0; q < NP; ++q) p[q] = (tdc_u2){a[q], b[q]};
}

// one operand of a 32-wide step in its parts
template <int NP>
struct tdc_op {
    tdc_h8 p[NP];
};

// a lane's operand from its shares of the two k-groups of a step
template <int NP>
__device__ __forceinline__ tdc_op<NP> tdc_split_op(tdc_f4 lo, tdc_f4 hi, const TdcScale &s)
{
    tdc_u2 a[NP], b[NP];
    tdc_split4<NP>(lo, s, a);
    tdc_split4<NP>(hi, s, b);
    tdc_op<NP> o;
#pragma unroll
    for (int i = 0; i < NP; ++i) o.p[i] = __builtin_bit_cast(tdc_h8, (tdc_u4){a[i][0], a[i][1], b[i][0], b[i][1]});
    return o;
}

constexpr int TDC_LEVELS = 2;
// whether the parts of weights are lifted
constexpr bool tdc_lift_weights(int np) { return np == 2; }

// The products of a step, the smallest first, each with its level and the weights' and the activations' part.
template <int NP>
struct TdcProducts;
template <>
struct TdcProducts<2> {
    static constexpr int N = 3, level[3] = {1, 1, 0}, w[3] = {1, 0, 0}, x[3] = {0, 1, 0};
};
template <>
struct TdcProducts<3> {
    static constexpr int N = 6, level[6] = {0, 1, 1, 1, 0, 0}, w[6] = {2, 1, 0, 0, 1, 0}, x[6] = {0, 1, 2, 1, 0, 0};
};

// SWAP: D's rows are the pixels
template <int NP, bool SWAP = false>
__device__ __forceinline__ tdc_f4 tdc_mfma_part(int i, const tdc_h8 (&w)[NP], const tdc_h8 (&x)[NP], tdc_f4 c)
{
    const int iw = TdcProducts<NP>::w[i], ix = TdcProducts<NP>::x[i];
    return SWAP ? __builtin_amdgcn_mfma_f32_16x16x32_f16(x[ix], w[iw], c, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x32_f16(w[iw], x[ix], c, 0, 0, 0);
}

// accumulators of the levels -> the sum
__device__ __forceinline__ tdc_f4 tdc_levels(const tdc_f4 (&acc)[TDC_LEVELS])
{
    tdc_f4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fmaf(acc[1][i], 0x1p-11f, acc[0][i]);
    return v;
}

__device__ __forceinline__ tdc_f4 tdc_ldexp4(tdc_f4 v, int e) { return (tdc_f4){ldexpf(v[0], e), ldexpf(v[1], e), ldexpf(v[2], e), ldexpf(v[3], e)}; }

// Largest magnitude, NaN if one is (v_maximum3_f32: two values an instruction).
__device__ __forceinline__ float tdc_largest(float m, tdc_f4 v)
{
    m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, fabsf(v[0])), fabsf(v[1]));
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, fabsf(v[2])), fabsf(v[3]));
}
// max(a, |b|, |c|) of those that are no NaN.  Asm: fmaxf would take an instruction more for each that might be a signalling NaN.  b and
// c must not come from the matrix cores directly (see tdc_split2).
__device__ __forceinline__ float tdc_max3_abs(float a, float b, float c)
{
    float m;
    asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(m) : "v"(a), "v"(b), "v"(c));
    return m;
}
// Largest magnitude of those that are numbers.
__device__ __forceinline__ float tdc_largest_number(float m, tdc_f4 v) { return fmaxf(fmaxf(fmaxf(m, fabsf(v[0])), fmaxf(fabsf(v[1]), fabsf(v[2]))), fabsf(v[3])); }
// The smallest of several magnitudes that is not zero, as an integer: start with ~0u.
__device__ __forceinline__ unsigned tdc_smallest(unsigned s, float m) { return min(s, __builtin_bit_cast(unsigned, m) - 1u); }
__device__ __forceinline__ bool tdc_is_small(unsigned s, float limit) { return s < __builtin_bit_cast(unsigned, limit) - 1u; }
__device__ __forceinline__ bool tdc_any_lane(bool b) { return __builtin_amdgcn_ballot_w64(b) != 0; }
__device__ __forceinline__ bool tdc_finite(float m) { return m < INFINITY; }

// the largest over the four lane groups that hold a pixel's channels, for lanes that hold one pixel each
__device__ __forceinline__ float tdc_pixel_max(float m)
{
    const unsigned u = __builtin_bit_cast(unsigned, m);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned v = max(a[0], a[1]);             // magnitudes compare as integers, a NaN above all
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return __builtin_bit_cast(float, max(b[0], b[1]));
}

// what the lane eight further in a row of 16 holds
__device__ __forceinline__ int tdc_row_ror8(int v) { return __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true); }

// the largest of a wavefront, as bits, in a scalar register
__device__ __forceinline__ unsigned tdc_wave_max(float m)
{
    unsigned u = __builtin_bit_cast(unsigned, tdc_pixel_max(m));
    u = max(u, (unsigned)__builtin_amdgcn_mov_dpp((int)u, 0x128, 0xf, 0xf, true));      // row_ror:8
    u = max(u, (unsigned)__builtin_amdgcn_mov_dpp((int)u, 0x124, 0xf, 0xf, true));      // row_ror:4
    u = max(u, (unsigned)__builtin_amdgcn_mov_dpp((int)u, 0x122, 0xf, 0xf, true));      // row_ror:2
    u = max(u, (unsigned)__builtin_amdgcn_mov_dpp((int)u, 0x121, 0xf, 0xf, true));      // row_ror:1
    return (unsigned)__builtin_amdgcn_readfirstlane((int)u);
}

// Exponent of the power of two that takes a magnitude (its bits) to 2^target .. 2^(target+1); `other` where it says nothing.
__device__ __forceinline__ int tdc_scale_of(unsigned bits, int target, int other)
{
    const int e = (int)(bits >> 23);
    return e == 0 || e >= 255 ? other : min(target + 127 - e, 100);
}
constexpr int TDC_X_TARGET = 6, TDC_X_OTHER = 6, TDC_Z2_TARGET = 12;
constexpr int TDC_LOWEST = -13;      // scaled values from 2^TDC_LOWEST on keep all their bits
constexpr int tdc_lowest_weight(int np) { return tdc_lift_weights(np) ? TDC_LOWEST : -1; }
constexpr float TDC_FP16_MAX = 65504.f;
// Exponents of the channels of weights that are kept out of the parts, which are NaN, and of output channels without a weight that is
// not 0.  The latter have weights of 2^12 and 2^13 in parts, so that their sums are of the usual size and no stage need know
// them; the exponent then makes them 0.
constexpr int TDC_WIDE = 1 << 20, TDC_EMPTY = 1 << 21;

// k-group kg's share of a lane's fp32 weights of 16-channel block `block` (layout: tdc_internal.h)
__device__ __forceinline__ tdc_f4 tdc_raw_weights(tdc_rsrc r, int block, int k_groups, int kg, int lane)
{
    return tdc_buf_load4(r, ((unsigned)(block * k_groups + kg) * 64u + lane) * 16u);
}
// ... which lie behind the parts and the exponents
__device__ __forceinline__ const char *tdc_raw_base(const void *parts, unsigned parts_bytes, int m_blocks) { return static_cast<const char *>(parts) + parts_bytes + 64u * m_blocks; }

// What some factors hold: whether the NaNs among their sums can only come from NaNs among them.
struct TdcFactors {
    float largest = 0.f;       // magnitude of the largest that is not NaN
    bool nan = false;
    __device__ __forceinline__ void see(tdc_f4 v)
    {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            nan |= v[j] != v[j];
            largest = fmaxf(largest, fabsf(v[j]));
        }
    }
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

#endif
