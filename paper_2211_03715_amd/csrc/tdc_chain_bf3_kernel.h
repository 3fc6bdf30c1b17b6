// CHAIN on the bf16 matrix cores: the three stages of one output tile in one launch, as in tdc_chain_kernel.h, every fp32
// factor in three bf16 parts (tdc_bf3.h).  For layers whose three sums are short (tdc_chain3_bf3): there it is the more accurate form, and
// with no scale to find before the first product the faster one; the figures of longer sums below are from before those went to
// two fp16 parts (tdc_chain3_kernel.h).
//
//   stage 1   units of PB1 pixel blocks x MB1 channel blocks; x goes from memory into registers one step ahead, is split
//             there, and the finished z1 values are split once more and stored as parts: 8-byte LDS cells of four channels,
//             [part][channel block][lane group][pixel], which any pair of k-groups of stage 2 reads as operand halves;
//   stage 2   a wavefront computes all R2 channels (NB2 blocks) of PB pixel blocks, weights streamed one step ahead;
//   stage 3   its operand is the accumulators, split in registers; weights streamed one output block ahead.
// A tile of one or two groups of pixel blocks has fewer groups than the workgroup has wavefronts: four or two of them then
// share a group, each with a slice of stage 2's contraction; the partial sums meet in LDS and every wavefront goes on with all
// of z2 and its share of the output blocks.
//
// What bounds it.  The fp32 form was bound by the fp32 matrix rate plus the phases of its one resident workgroup, which do
// not overlap: 32 -> 32 ranks, 128 channels at 28x28, batch 256: 97 us, of which 45 us are matrix cycles and 39 us compulsory
// bytes.  Here the products take 3/8 of the cycles, and workgroups are four wavefronts on tiles of at most 128 pixels, so that
// two to three share a compute unit and one's loads run under another's products: 77 us (62 us where x and y of consecutive
// calls are the same buffers); 64 -> 32 ranks, 64 channels at 224x224: 35.7 -> 27.0 us.  What is left is memory, with loads
// one step ahead.  The weight fragments come through the L1 at 54 bytes a cycle: PB pixel blocks share one.  PB = 4 halves that
// traffic and needs 144 to 256 registers instead of 99 to 256 (three z2 blocks in NCHW spill 19 to 22).  The selector offers
// PB = 2 alone; with the buffers of a call in cache an exhaustive search takes PB = 4 on larger tiles in three of sixteen cases
// (128 channels at 28x28, ranks 32, batch 128: 36.8 -> 31.4 us), with new buffers per call it was 2 to 10 % slower.
// With few pixels (24 per compute unit) a workgroup has its compute unit to itself and the chain of its steps is the time;
// sharing cuts it: ranks 80, 256 channels at 14x14, batch 32: 34.6 us unshared, 20.7 shared (fp32 FUSED: 33.0).
#ifndef TDC_CHAIN_BF3_KERNEL_H
#define TDC_CHAIN_BF3_KERNEL_H

#include <type_traits>

#include "tdc_bf3.h"
#include "tdc_internal.h"
#include "tdc_stage1.h"

constexpr int TDC_CHAIN_BF3_WAVES = 4;

struct TdcChainBf3Args {
    const float *x;
    const void *uin3, *core3, *uout3;
    float *y;
    TdcEpi epi;
    int C, N, H, W, Ho, Wo, K, stride, pad;
    int NB1, NB3, S1, KG2, S2;                 // channel blocks; 32-wide steps of stage 1; k-groups and steps of stage 2
    int TH, TW, QH, QW, Q, P, QB, n_pg2;
    int lg_ks;                                 // log2 of the wavefronts that share a group of pixel blocks (tdc_chain3_share)
    int pitch1;                                // LDS row pitch of the z1 tile, in 8-byte cells
    int RPR, n_pg1, n_mg1;                     // runs per tile row; pixel groups and channel groups of stage 1
    int tiles_x, tiles, xcd_per, xcd_rem;
    int vec;                                   // NCHW: y goes out in 16-byte quads of pixels
    unsigned uin_bytes, core_bytes, uout_bytes;
    TdcDiv div_tiles_x, div_tiles, div_QW, div_TW, div_RPR, div_mg1, div_NB1, div_K;
};

namespace {

// Stage 1 for the workgroup.  RUNS: a lane owns runs of four consecutive pixels (see TdcStage1R), a unit is 16 runs.
template <int LAY, int MB1>
struct ChainBf3Stage1 {
    static constexpr bool RUNS = LAY == TDC_LAY_NCHW_RUNS, NHWC = LAY == TDC_LAY_NHWC;
    static constexpr int PB = RUNS ? 4 : 2;
    static constexpr int NR = RUNS ? 8 : 2 * PB;      // 16-byte registers of x per step
    const TdcChainBf3Args &a;
    tdc_rsrc xrs, urs;
    int lane, g, l16, wave, h0, w0, wa, n_units;
    int fu, fs, fmg;                                   // fetch cursor: unit, step, channel group of the unit
    unsigned xoff[RUNS ? 1 : PB];
    float largest = 0.f;                               // magnitude of this lane's largest z1 value, NaN if there is one
    unsigned smallest = ~0u;                           // of its pixels' largest values the smallest (tdc_smallest)

    __device__ __forceinline__ ChainBf3Stage1(const TdcChainBf3Args &args, int lane_, int wave_, int b, int h0_, int w0_) : a(args)
    {
        lane = lane_; g = lane >> 4; l16 = lane & 15; wave = wave_; h0 = h0_; w0 = w0_;
        wa = w0 > 0 ? (w0 & ~3) : 0;
        const int HW = a.H * a.W;
        xrs = tdc_make_rsrc(a.x + (size_t)b * a.C * HW, (unsigned)a.C * HW * 4u);
        urs = tdc_make_rsrc(a.uin3, a.uin_bytes);
        n_units = a.n_pg1 * a.n_mg1;
        fu = wave;
        place();
    }
    __device__ __forceinline__ void place()
    {
        fs = 0;
        const bool live = fu < n_units;
        const int pg = live ? tdc_div(fu, a.div_mg1) : 0;
        fmg = live ? fu - pg * a.n_mg1 : 0;
#pragma unroll
        for (int pb = 0; pb < (RUNS ? 1 : PB); ++pb) {
            bool ok;
            int h, w;
            if (RUNS) {
                const int rho = 16 * pg + l16, qh = tdc_div(rho, a.div_RPR);
                h = h0 + qh;
                w = wa + 4 * (rho - qh * a.RPR);
                ok = qh < a.QH;
            } else {
                const int q = 16 * (pg * PB + pb) + l16, qh = tdc_div(q, a.div_QW);
                h = h0 + qh;
                w = w0 + q - qh * a.QW;
                ok = q < a.Q;
            }
            ok = ok & live & ((unsigned)h < (unsigned)a.H) & ((unsigned)w < (unsigned)a.W);   // no branches in the pipeline
            xoff[pb] = ok ? (unsigned)(h * a.W + w) * (NHWC ? 4u * a.C : 4u) : TDC_OOB;
        }
    }
    // channels past C read 0: in NCHW they lie beyond the image's descriptor by themselves
    __device__ __forceinline__ void fetch(tdc_f4 (&x)[NR], tdc_op3 (&w)[MB1])
    {
        const unsigned dead = fu < n_units ? 0u : TDC_OOB;
        const unsigned HW4 = (unsigned)(a.H * a.W) * 4u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = 32 * fs + 16 * h + 4 * g;
            if (RUNS) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    x[4 * h + j] = tdc_buf_load4(xrs, ((unsigned)(c + j) * HW4 + xoff[0]) | (xoff[0] & TDC_OOB));
            } else {
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    if (NHWC) {
                        x[2 * pb + h] = tdc_buf_load4(xrs, (xoff[pb] + 4u * c) | (c < a.C ? 0u : TDC_OOB) | (xoff[pb] & TDC_OOB));
                    } else {
                        const unsigned o = ((unsigned)c * HW4 + xoff[pb]) | (xoff[pb] & TDC_OOB);
                        x[2 * pb + h] = (tdc_f4){tdc_buf_load(xrs, o), tdc_buf_load(xrs, o + HW4), tdc_buf_load(xrs, o + 2u * HW4), tdc_buf_load(xrs, o + 3u * HW4)};
                    }
                }
            }
        }
#pragma unroll
        for (int mb = 0; mb < MB1; ++mb) {
            const int blk = fmg * MB1 + mb;
            const unsigned o = ((unsigned)(blk * a.S1 + fs) * 3072u + lane * 16u) | dead | (blk < a.NB1 ? 0u : TDC_OOB);
#pragma unroll
            for (int q = 0; q < 3; ++q) w[mb].p[q] = __builtin_bit_cast(tdc_bf8, tdc_buf_load4(urs, o + q * 1024u));
        }
        if (++fs == a.S1) {
            fu += TDC_CHAIN_BF3_WAVES;
            place();
        }
    }
    // tile cells whose image column is outside [0, W): the runs never produce them
    __device__ __forceinline__ void zero_outside(tdc_u2 *__restrict__ z1s) const
    {
        if (!RUNS) return;
        const int left = max(-w0, 0), right = max(w0 + a.QW - a.W, 0);
        const int per_row = left + right, total = per_row * a.QH * 12 * a.NB1;
        for (int e = 64 * wave + lane; e < total; e += 64 * TDC_CHAIN_BF3_WAVES) {
            const int c = e % per_row, r = (e / per_row) % a.QH, pl = e / (per_row * a.QH);
            const int qw = c < left ? c : a.QW - right + (c - left);
            z1s[pl * a.pitch1 + r * a.QW + qw] = (tdc_u2){0u, 0u};
        }
    }
    __device__ __forceinline__ void multiply(tdc_f4 (&acc)[MB1][PB], const tdc_f4 (&x)[NR], const tdc_op3 (&w)[MB1]) const
    {
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            tdc_op3 b;
            if (RUNS)
                b = tdc_split_op((tdc_f4){x[0][pb], x[1][pb], x[2][pb], x[3][pb]},
                                 (tdc_f4){x[4 % NR][pb], x[5 % NR][pb], x[6 % NR][pb], x[7 % NR][pb]});
            else
                b = tdc_split_op(x[(2 * pb) % NR], x[(2 * pb + 1) % NR]);
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int mb = 0; mb < MB1; ++mb) acc[mb][pb] = tdc_mfma_bf(w[mb].p[TDC_BF3_A[i]], b.p[TDC_BF3_B[i]], acc[mb][pb]);
        }
    }
    // RAW: for sums some of which have no three parts
    template <bool RAW>
    __device__ __forceinline__ void store(tdc_u2 *__restrict__ z1s, int unit, const tdc_f4 (&acc)[MB1][PB]) const
    {
        const int pg = tdc_div(unit, a.div_mg1), mg = unit - pg * a.n_mg1;
        const int rho = 16 * pg + l16, qh = RUNS ? tdc_div(rho, a.div_RPR) : 0;
        const int qw0 = RUNS ? wa + 4 * (rho - qh * a.RPR) - w0 : 0;
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            const bool ok = RUNS ? qh < a.QH && qw0 + pb >= 0 && qw0 + pb < a.QW : pg * PB + pb < a.QB;
            const int pix = RUNS ? qh * a.QW + qw0 + pb : 16 * (pg * PB + pb) + l16;
#pragma unroll
            for (int mb = 0; mb < MB1; ++mb) {
                const int blk = mg * MB1 + mb;
                tdc_u2 p[3];
                if (RAW) tdc_split4_raw(acc[mb][pb], 0x1p-110f, p[0], p[1], p[2]);
                else tdc_split4(acc[mb][pb], p[0], p[1], p[2]);
                if (ok && blk < a.NB1) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) z1s[((q * a.NB1 + blk) * 4 + g) * a.pitch1 + pix] = p[q];
                }
            }
        }
    }
    __device__ __forceinline__ void run(tdc_u2 *__restrict__ z1s)
    {
        tdc_f4 x0[NR], x1[NR], acc[MB1][PB];
        tdc_op3 wa0[MB1], wa1[MB1];
        fetch(x0, wa0);
        zero_outside(z1s);
        const int total = wave < n_units ? (n_units - wave + TDC_CHAIN_BF3_WAVES - 1) / TDC_CHAIN_BF3_WAVES * a.S1 : 0;
        int unit = wave, step = 0;
        const auto clear = [&]() {
#pragma unroll
            for (int mb = 0; mb < MB1; ++mb)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) acc[mb][pb] = tdc_f4_zero();
        };
        const auto done = [&]() {
            if (++step < a.S1) return;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                float m = 0.f;
#pragma unroll
                for (int mb = 0; mb < MB1; ++mb) m = tdc_largest(m, acc[mb][pb]);
                largest = __builtin_elementwise_maximum(largest, m);
                smallest = tdc_smallest(smallest, m);
            }
            store<false>(z1s, unit, acc);
            unit += TDC_CHAIN_BF3_WAVES;
            step = 0;
            clear();
        };
        clear();
        for (int i = 0; i < total; i += 2) {
            fetch(x1, wa1);
            multiply(acc, x0, wa0);
            done();
            fetch(x0, wa0);
            if (i + 1 < total) {
                multiply(acc, x1, wa1);
                done();
            }
        }
    }
    // The wavefront's units once more in fp32, one load at a time (see tdc_bf3.h); those whose NaNs are x's or the weights' stay.
    __device__ __forceinline__ void redo(tdc_u2 *__restrict__ z1s, bool small)
    {
        tdc_f4 x[NR];
        tdc_op3 w[MB1];
        const auto join = [&](int mb, int h) {
            tdc_u2 p[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const tdc_u4 u = __builtin_bit_cast(tdc_u4, w[mb].p[q]);
                p[q] = h ? (tdc_u2){u[2], u[3]} : (tdc_u2){u[0], u[1]};
            }
            return tdc_join4(p);
        };
        for (int unit = wave; unit < n_units; unit += TDC_CHAIN_BF3_WAVES) {
            TdcFactors seen;
            fu = unit;
            place();
            for (int i = 0; i < a.S1; ++i) {
                fetch(x, w);
#pragma unroll
                for (int j = 0; j < NR; ++j) seen.see(x[j]);
#pragma unroll
                for (int mb = 0; mb < MB1; ++mb) {
                    const tdc_u4 u = __builtin_bit_cast(tdc_u4, w[mb].p[0]);
                    seen.see((tdc_u2){u[0], u[1]});
                    seen.see((tdc_u2){u[2], u[3]});
                }
            }
            if (!small && seen.explain_nan()) continue;
            tdc_f4 acc[MB1][PB];
#pragma unroll
            for (int mb = 0; mb < MB1; ++mb)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) acc[mb][pb] = tdc_f4_zero();
            fu = unit;
            place();
            for (int i = 0; i < a.S1; ++i) {
                fetch(x, w);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int mb = 0; mb < MB1; ++mb) {
                        const tdc_f4 wh = join(mb, h);
#pragma unroll
                        for (int j = 0; j < 4; ++j)
#pragma unroll
                            for (int pb = 0; pb < PB; ++pb)
                                acc[mb][pb] = tdc_mfma(wh[j], RUNS ? x[(4 * h + j) % NR][pb] : x[(2 * pb + h) % NR][j], acc[mb][pb]);
                    }
            }
            store<true>(z1s, unit, acc);
        }
    }
};

// The image and the tile of this workgroup: one contiguous range of (image, tile) pairs per XCD, so that halos are shared
// within its L2.
struct ChainBf3Tile {
    int b, i0, j0;
    __device__ __forceinline__ ChainBf3Tile(const TdcChainBf3Args &a)
    {
        const int lin = blockIdx.y * a.tiles + blockIdx.x, xcd = lin & 7, slot = lin >> 3;
        const int lb = xcd * a.xcd_per + min(xcd, a.xcd_rem) + slot;
        b = tdc_div(lb, a.div_tiles);
        const int tile = lb - b * a.tiles, ty = tdc_div(tile, a.div_tiles_x), tx = tile - ty * a.tiles_x;
        i0 = ty * a.TH;
        j0 = tx * a.TW;
    }
};

// z1 cells of the (0, 0) tap of pixel l16 of each block of a group
template <int PB>
__device__ __forceinline__ void chain_bf3_z1_base(const TdcChainBf3Args &a, int group, int lane, int (&qbase)[PB])
{
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        const int p = 16 * (group * PB + pb) + (lane & 15);
        const int ph = tdc_div(p, a.div_TW), pw = p - ph * a.TW;
        qbase[pb] = (lane >> 4) * a.pitch1 + (p < a.P ? ph * a.stride * a.QW + pw * a.stride : 0);
    }
}

// The outputs of a group of pixel blocks.
template <int PB, bool NHWC>
struct ChainBf3Out {
    const TdcChainBf3Args &a;
    int g, l16, b, P2;
    tdc_rsrc yrs;
    unsigned yq[PB][4];      // NCHW: byte offset of pixel 4*g + i of block pb in one channel plane, or TDC_OOB
    int ypix[PB];            // NHWC: index of pixel l16 of block pb in the output image, or -1

    __device__ __forceinline__ ChainBf3Out(const TdcChainBf3Args &args, const ChainBf3Tile &at, int group, int lane) : a(args)
    {
        g = lane >> 4; l16 = lane & 15; b = at.b;
        P2 = a.Ho * a.Wo;
        yrs = tdc_make_rsrc(a.y + (size_t)b * a.N * P2, (unsigned)a.N * P2 * 4u);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = 16 * (group * PB + pb) + 4 * g + i;
                const int ph = tdc_div(p, a.div_TW), pw = p - ph * a.TW;
                const int oi = at.i0 + ph, oj = at.j0 + pw;
                yq[pb][i] = (p < a.P && oi < a.Ho && oj < a.Wo) ? (unsigned)(oi * a.Wo + oj) * 4u : TDC_OOB;
            }
            const int p = 16 * (group * PB + pb) + l16;
            const int ph = tdc_div(p, a.div_TW), pw = p - ph * a.TW;
            const int oi = at.i0 + ph, oj = at.j0 + pw;
            ypix[pb] = (p < a.P && oi < a.Ho && oj < a.Wo) ? oi * a.Wo + oj : -1;
        }
    }
    // sums of output block nb, through the epilogue
    template <bool EPI>
    __device__ __forceinline__ void put(int nb, tdc_f4 (&acc3)[PB]) const
    {
        if (NHWC) {
            const int n = 16 * nb + 4 * g;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
                if (ypix[pb] >= 0 && n < a.N) {
                    const size_t cell = ((size_t)b * P2 + ypix[pb]) * a.N + n;
                    if constexpr (EPI) tdc_store_nhwc<true>(a.y, a.epi, acc3[pb], n, cell);
                    else tdc_store4_stream(reinterpret_cast<tdc_f4 *>(a.y + cell), acc3[pb]);
                }
            return;
        }
        // channels past N lie beyond the descriptor: the hardware drops those stores
        const unsigned row = (unsigned)(16 * nb + l16) * P2 * 4u;
        if constexpr (EPI) {
            const int n = 16 * nb + l16;
            const float bias = (a.epi.bias && n < a.N) ? a.epi.bias[n] : 0.f;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float v = acc3[pb][i] + bias;
                    if (a.epi.residual && n < a.N && !(yq[pb][i] & TDC_OOB))
                        v += a.epi.residual[(size_t)b * a.N * P2 + (size_t)n * P2 + (yq[pb][i] >> 2)];
                    acc3[pb][i] = a.epi.relu ? fmaxf(v, 0.f) : v;
                }
        }
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            if (a.vec) {
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, acc3[pb]), yrs, (int)((row + yq[pb][0]) | (yq[pb][0] & TDC_OOB)), 0, 0);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = acc3[pb][i];   // a copy: __builtin_bit_cast of a vector element reads element 0
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), yrs, (int)((row + yq[pb][i]) | (yq[pb][i] & TDC_OOB)), 0, 0);
                }
            }
        }
    }
};

// Stages 2 and 3 of a group once more in fp32, one load at a time (see tdc_bf3.h), unless its NaNs are z1's or the weights'.
template <int NB2, int PB, int LAY>
__device__ __forceinline__ void chain_bf3_redo(const TdcChainBf3Args &a, const tdc_u2 *__restrict__ z1s, int group, int lane, int slice)
{
    constexpr bool NHWC = LAY == TDC_LAY_NHWC;
    constexpr int S3 = (NB2 + 1) / 2;
    const tdc_rsrc crs = tdc_make_rsrc(a.core3, a.core_bytes), ors = tdc_make_rsrc(a.uout3, a.uout_bytes);
    int qbase[PB];
    chain_bf3_z1_base<PB>(a, group, lane, qbase);
    const auto cell_of = [&](int kg) {
        const int tap = tdc_div(kg, a.div_NB1), r = tdc_div(tap, a.div_K);
        return (kg - tap * a.NB1) * 4 * a.pitch1 + r * a.QW + tap - r * a.K;
    };
    const auto z1_at = [&](int cell, int pb) {
        tdc_u2 u[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) u[q] = z1s[q * a.NB1 * 4 * a.pitch1 + cell + qbase[pb]];
        return tdc_join4(u);
    };
    TdcFactors seen;
    for (int kg = 0; kg < a.KG2; ++kg) {
        const int cell = cell_of(kg);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) seen.see(z1s[cell + qbase[pb]]);
#pragma unroll
        for (int mb = 0; mb < NB2; ++mb) seen.see(tdc_first_parts(crs, mb, a.S2, kg, lane));
    }
    for (int nb = 0; nb < a.NB3; ++nb)
#pragma unroll
        for (int kg = 0; kg < NB2; ++kg) seen.see(tdc_first_parts(ors, nb, S3, kg, lane));
    if (seen.explain_nan() && !tdc_any_lane(seen.low)) return;     // and z2 cannot be small

    tdc_f4 z2[NB2][PB];
#pragma unroll
    for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) z2[mb][pb] = tdc_f4_zero();
    for (int kg = 0; kg < a.KG2; ++kg) {
        const int cell = cell_of(kg);
        tdc_f4 z[PB];
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) z[pb] = z1_at(cell, pb);
#pragma unroll
        for (int mb = 0; mb < NB2; ++mb) {
            const tdc_f4 w = tdc_join_weights(crs, mb, a.S2, kg, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) z2[mb][pb] = tdc_mfma(w[j], z[pb][j], z2[mb][pb]);
        }
    }
    __threadfence();         // the outputs stored before are in place, these follow them
    const ChainBf3Out<PB, NHWC> out(a, ChainBf3Tile(a), group, lane);
    for (int nb = slice; nb < a.NB3; nb += 1 << a.lg_ks) {
        tdc_f4 acc3[PB];
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc3[pb] = tdc_f4_zero();
#pragma unroll
        for (int kg = 0; kg < NB2; ++kg) {
            const tdc_f4 w = tdc_join_weights(ors, nb, S3, kg, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
                    acc3[pb] = NHWC ? tdc_mfma(w[j], z2[kg][pb][j], acc3[pb]) : tdc_mfma(z2[kg][pb][j], w[j], acc3[pb]);
        }
        out.template put<true>(nb, acc3);
    }
}

// Wavefronts per SIMD an instance has registers for; the rarely run code must not cost one.
constexpr int chain_bf3_wavefronts(int nb2, int pb, int lay, int mb1)
{
    if (pb > 2) return 2;
    if (nb2 <= 2) return lay == TDC_LAY_NCHW_RUNS ? 5 - mb1 : mb1 <= 2 ? 4 : 3;
    return nb2 == 3 && lay == TDC_LAY_NHWC ? 3 : 2;
}

template <int NB2, int PB, int LAY, int MB1>
__global__ __launch_bounds__(64 * TDC_CHAIN_BF3_WAVES, chain_bf3_wavefronts(NB2, PB, LAY, MB1)) void tdc_chain_bf3_kernel(TdcChainBf3Args a)
{
    constexpr bool NHWC = LAY == TDC_LAY_NHWC;
    extern __shared__ tdc_u2 z1s[];                              // [3 parts][NB1][4][pitch1], then the partial sums of ks > 1
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const auto stage1 = [&](const TdcChainBf3Args &args) {
        const ChainBf3Tile t(args);
        return ChainBf3Stage1<LAY, MB1>(args, lane, wave, t.b, t.i0 * args.stride - args.pad, t.j0 * args.stride - args.pad);
    };
    {
        ChainBf3Stage1<LAY, MB1> s1 = stage1(a);
        s1.run(z1s);
        // a value without three parts among x, the weights or z1 itself, or a pixel of nothing but small ones
        if (__builtin_expect(tdc_any_lane(!(s1.largest < TDC_BIG) || tdc_is_small(s1.smallest)), 0))
            stage1(tdc_args_again<TdcChainBf3Args>()).redo(z1s, tdc_any_lane(tdc_is_small(s1.smallest)));
    }
    const ChainBf3Tile at(a);
    __syncthreads();

    const int plane = a.NB1 * 4 * a.pitch1;                      // cells of one part
    const tdc_rsrc crs = tdc_make_rsrc(a.core3, a.core_bytes);
    const tdc_rsrc ors = tdc_make_rsrc(a.uout3, a.uout_bytes);
    // with fewer groups than wavefronts 2 or 4 of them share one: each takes a slice of stage 2's contraction, the sums meet in
    // LDS, and each takes every ks-th output block of stage 3 (the loop then runs once for every wavefront)
    const int ks = 1 << a.lg_ks, slice = wave & (ks - 1);
    for (int pg = wave >> a.lg_ks; pg < a.n_pg2; pg += TDC_CHAIN_BF3_WAVES) {
        // ---- stage 2: z2 channels 16*mb + 4*g + {0..3} of pixel l16 of block pb
        int qbase[PB];
        chain_bf3_z1_base<PB>(a, pg, lane, qbase);
        tdc_f4 acc2[NB2][PB];
#pragma unroll
        for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) acc2[mb][pb] = tdc_f4_zero();
        {
            // a fetch past the last step stays inside the descriptor or reads 0, and is never multiplied
            const auto fetch_w = [&](int step, tdc_op3(&w)[NB2]) {
#pragma unroll
                for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        w[mb].p[q] = __builtin_bit_cast(tdc_bf8, tdc_buf_load4(crs, (unsigned)(mb * a.S2 + step) * 3072u + q * 1024u + lane * 16u));
            };
            const int st0 = slice * a.S2 >> a.lg_ks, st1 = (slice + 1) * a.S2 >> a.lg_ks;
            // next k-group: tap offset toff = r*QW + s, channel block dg
            int kg = 2 * st0;
            const int tap = tdc_div(kg, a.div_NB1), r = tdc_div(tap, a.div_K);
            int dg = kg - tap * a.NB1, s = tap - r * a.K, toff = r * a.QW + s;
            const auto next_cell = [&]() {
                const int cell = dg * 4 * a.pitch1 + toff;
                const bool w1 = dg + 1 == a.NB1;
                dg = w1 ? 0 : dg + 1;
                const int ns = s + (w1 ? 1 : 0);
                const bool w2 = ns == a.K;
                s = w2 ? 0 : ns;
                toff += (w1 ? 1 : 0) + (w2 ? a.QW - a.K : 0);
                ++kg;
                return cell;
            };
            const auto step2 = [&](const tdc_op3(&w)[NB2]) {
                const int lo = next_cell();
                const bool whole = kg < a.KG2;                   // else the last half step, whose weights are zero: any finite cell does
                const int nx = next_cell(), hi = whole ? nx : lo;
                const auto read = [&](int pb) {
                    tdc_op3 o;
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const tdc_u2 u = z1s[q * plane + lo + qbase[pb]], v = z1s[q * plane + hi + qbase[pb]];
                        o.p[q] = __builtin_bit_cast(tdc_bf8, (tdc_u4){u[0], u[1], v[0], v[1]});
                    }
                    return o;
                };
                tdc_op3 bb[2];
                bb[0] = read(0);
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    if (pb + 1 < PB) bb[(pb + 1) & 1] = read(pb + 1);
#pragma unroll
                    for (int i = 0; i < 6; ++i)
#pragma unroll
                        for (int mb = 0; mb < NB2; ++mb)
                            acc2[mb][pb] = tdc_mfma_bf(w[mb].p[TDC_BF3_A[i]], bb[pb & 1].p[TDC_BF3_B[i]], acc2[mb][pb]);
                }
            };
            tdc_op3 wv0[NB2], wv1[NB2];
            fetch_w(st0, wv0);
            for (int st = st0; st < st1; st += 2) {
                fetch_w(st + 1, wv1);
                step2(wv0);
                fetch_w(st + 2, wv0);
                if (st + 1 < st1) step2(wv1);
            }
        }
        if (ks > 1) {      // partial sums, added in the order of the slices
            tdc_f4 *__restrict__ red = reinterpret_cast<tdc_f4 *>(z1s + 3 * plane);
#pragma unroll
            for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) red[((wave * NB2 + mb) * PB + pb) * 64 + lane] = acc2[mb][pb];
            __syncthreads();
            const int first = wave - slice;
#pragma unroll
            for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    tdc_f4 v = red[((first * NB2 + mb) * PB + pb) * 64 + lane];
                    for (int j = 1; j < ks; ++j) v += red[(((first + j) * NB2 + mb) * PB + pb) * 64 + lane];
                    acc2[mb][pb] = v;
                }
        }
        // ---- stage 3, operands swapped in NCHW: D[pixel 4*g + i][channel l16]; NHWC: D[channel 4*g + i][pixel l16]
        constexpr int S3 = (NB2 + 1) / 2;
        const auto fetch = [&](int nb, tdc_op3(&u)[S3]) {
#pragma unroll
            for (int st = 0; st < S3; ++st)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    u[st].p[q] = __builtin_bit_cast(tdc_bf8, tdc_buf_load4(ors, (unsigned)(nb * S3 + st) * 3072u + q * 1024u + lane * 16u));
        };
        tdc_op3 u0[S3], u1[S3];
        fetch(slice, u0);                                        // under the splitting of z2
        float largest = 0.f;                                     // magnitude of the largest of z2 and y, NaN if there is one
        unsigned smallest = ~0u;                                 // of the pixels' largest z2 values the smallest
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            float m = 0.f;
#pragma unroll
            for (int mb = 0; mb < NB2; ++mb) m = tdc_largest(m, acc2[mb][pb]);
            largest = __builtin_elementwise_maximum(largest, m);
            smallest = tdc_smallest(smallest, m);
        }
        largest = tdc_is_small(smallest) ? INFINITY : largest;
        asm("" : "+v"(largest));                                 // now: not behind the outputs, with all of acc2 kept until then
        tdc_op3 zb[S3][PB];
#pragma unroll
        for (int st = 0; st < S3; ++st)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) zb[st][pb] = tdc_split_op(acc2[2 * st][pb], 2 * st + 1 < NB2 ? acc2[(2 * st + 1) % NB2][pb] : tdc_f4_zero());
        const ChainBf3Out<PB, NHWC> out(a, at, pg, lane);
        // two instances of the loop, as in tdc_chain_kernel.h: without epilogue loads nothing ever waits for the stores
        const auto emit = [&](auto with_epi, int nb, const tdc_op3(&u)[S3]) {
            tdc_f4 acc3[PB];
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) acc3[pb] = tdc_f4_zero();
#pragma unroll
            for (int st = 0; st < S3; ++st)
#pragma unroll
                for (int i = 0; i < 6; ++i)
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb)
                        acc3[pb] = NHWC ? tdc_mfma_bf(u[st].p[TDC_BF3_A[i]], zb[st][pb].p[TDC_BF3_B[i]], acc3[pb])
                                        : tdc_mfma_bf(zb[st][pb].p[TDC_BF3_B[i]], u[st].p[TDC_BF3_A[i]], acc3[pb]);
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) largest = tdc_largest(largest, acc3[pb]);
            out.template put<decltype(with_epi)::value>(nb, acc3);
        };
        const auto stage3 = [&](auto with_epi) {
            for (int nb = slice; nb < a.NB3; nb += 2 * ks) {
                fetch(nb + ks, u1);
                emit(with_epi, nb, u0);
                fetch(nb + 2 * ks, u0);
                if (nb + ks < a.NB3) emit(with_epi, nb + ks, u1);
            }
        };
        if (a.epi.bias || a.epi.residual || a.epi.relu) stage3(std::true_type{});
        else stage3(std::false_type{});
        // a NaN, or z2 too large or too small for three parts: only then can an output be wrong
        if (__builtin_expect(tdc_any_lane(!(largest < TDC_BIG)), 0)) {
            int group = pg;
            asm volatile("" : "+s"(group));                      // its addresses are computed there, not kept from above
            chain_bf3_redo<NB2, PB, LAY>(tdc_args_again<TdcChainBf3Args>(), z1s, group, lane, slice);
        }
    }
}

}  // namespace

// (z2 blocks, pixel blocks of a unit) that have an instance: what fits 256 registers beside the weights in flight, or nearly
// so (three z2 blocks with PB = 4 in NCHW)
#define TDC_CHAIN_BF3_UNITS(X) X(1, 4) X(2, 4) X(3, 4) X(1, 2) X(2, 2) X(3, 2) X(4, 2) X(5, 2)

template <int LAY>
hipError_t tdc_launch_chain_bf3_lay(const TdcChainBf3Args &a, int nb2, int pb, int mb1, dim3 grid, size_t lds, hipStream_t s, bool prepare_only)
{
#define TDC_LAUNCH(N_, P_, M_)                                                                                    \
    if (mb1 == M_) {                                                                                              \
        hipError_t e = tdc_allow_lds((const void *)tdc_chain_bf3_kernel<N_, P_, LAY, M_>, lds);                       \
        if (e != hipSuccess || prepare_only) return e;                                                            \
        hipLaunchKernelGGL((tdc_chain_bf3_kernel<N_, P_, LAY, M_>), grid, dim3(64 * TDC_CHAIN_BF3_WAVES), lds, s, a); \
        return hipGetLastError();                                                                                 \
    }
#define TDC_X(N_, P_)                                                                                             \
    if (nb2 == N_ && pb == P_) {                                                                                  \
        TDC_LAUNCH(N_, P_, 1) TDC_LAUNCH(N_, P_, 2) TDC_LAUNCH(N_, P_, 3)                                         \
    }
    TDC_CHAIN_BF3_UNITS(TDC_X)
#undef TDC_X
#undef TDC_LAUNCH
    return hipErrorInvalidValue;
}

#endif
