// CHAIN on the fp16 matrix cores: the three stages of one output tile in one launch, as in tdc_chain_kernel.h, every fp32
// factor in two scaled fp16 parts (tdc_split.h).  Layers of short sums run on the bf16 ones (tdc_chain_bf3_kernel.h).
//
//   stage 1   units of PB1 pixel blocks x MB1 channel blocks; x goes from memory into registers one or two steps ahead, is
//             split there, and the finished z1 values are split once more and stored as parts: 8-byte LDS cells of four channels,
//             [part][channel block][lane group][pixel], which any pair of k-groups of stage 2 reads as operand halves;
//   stage 2   a wavefront computes all R2 channels (NB2 blocks) of PB pixel blocks; weights come through LDS in chunks that
//             all wavefronts share (Chain3Feed), or straight into registers one step ahead where each needs its own;
//   stage 3   its operand is the accumulators, split in registers; weights likewise, one output block ahead.
// A tile of one or two groups of pixel blocks has fewer groups than the workgroup has wavefronts: four or two of them then
// share a group, each with a slice of stage 2's contraction; the partial sums meet in LDS and every wavefront goes on with all
// of z2 and its share of the output blocks.
//
// What bounds it.  The fp32 form was bound by the fp32 matrix rate plus the phases of its one resident workgroup, which do
// not overlap: 32 -> 32 ranks, 128 channels at 28x28, batch 256: 97 us, of which 45 us are matrix cycles and 39 us compulsory
// bytes.  Here the products take 3/16 of the cycles (two parts), and workgroups are four wavefronts on tiles of at most 128
// pixels, so that two to three share a compute unit and one's loads run under another's products: 77 us with three bf16 parts and
// every wavefront's weights through the L1, 72.6 with two fp16 parts, 67.0 with shared weights and three workgroups to a
// compute unit; 64 -> 32 ranks, 64 channels at 224x224: 35.7 -> 27.0 -> 23.8 -> 22.5 us.  What is left is memory.  PB = 4
// halves the reads of weight fragments and needs about 1.5 times the registers; the selector offers PB = 2 alone: PB = 4 was 2 to
// 10 % slower with new buffers per call (three bf16 parts).
// With few pixels (24 per compute unit) a workgroup has its compute unit to itself and the chain of its steps is the time;
// sharing cuts it: ranks 80, 256 channels at 14x14, batch 32, three bf16 parts: 34.6 us unshared, 20.7 shared (fp32 FUSED: 33.0).
#ifndef TDC_CHAIN3_KERNEL_H
#define TDC_CHAIN3_KERNEL_H

#include <type_traits>

#include "tdc_split.h"
#include "tdc_internal.h"
#include "tdc_stage1.h"

constexpr int TDC_CHAIN3_WAVES = 4;

struct TdcChain3Args {
    const float *x;
    const void *uin, *core, *uout;             // in parts; core and uout with their exponents behind *_bytes
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
    int z1_exp;                                // z1 is kept 2^-z1_exp times its scaled sums
    unsigned uin_bytes, core_bytes, uout_bytes;
    TdcDiv div_tiles_x, div_tiles, div_QW, div_TW, div_RPR, div_mg1, div_NB1, div_K;
    int lost2, lost3;                          // what a channel's largest output must reach, see the launch
};

namespace {

constexpr int NP = 2;      // parts

// LDS: the largest magnitude each wavefront has loaded first (later what it has seen) and whether it wants the tile in fp32, then z1.
enum { CHAIN3_SMALL = 1, CHAIN3_NO_NUMBER = 2, CHAIN3_NAN = 1, CHAIN3_TOO_LARGE = 2 };
struct Chain3Shared {
    unsigned first[TDC_CHAIN3_WAVES], bad[TDC_CHAIN3_WAVES];
};

// x is multiplied by 2 to this
__device__ __forceinline__ int chain3_x_exp(const Chain3Shared &sh)
{
    const tdc_u4 first = *reinterpret_cast<const tdc_u4 *>(sh.first);
    return tdc_scale_of((unsigned)__builtin_amdgcn_readfirstlane((int)max(max(first[0], first[1]), max(first[2], first[3]))), TDC_X_TARGET, TDC_X_OTHER);
}

// Stage 1 for the workgroup.  RUNS: a lane owns runs of four consecutive pixels (see TdcStage1R), a unit is 16 runs.
template <int LAY, int MB1, bool DEEP>
struct Chain3Stage1 {
    static constexpr bool RUNS = LAY == TDC_LAY_NCHW_RUNS, NHWC = LAY == TDC_LAY_NHWC;
    static constexpr int PB = RUNS ? 4 : 2;
    static constexpr int NR = RUNS ? 8 : 2 * PB;      // 16-byte registers of x per step
    // Depth 1 in lean runs: three workgroups to a compute unit instead of two overlap more than a step on its way (128 channels at
    // 28x28, ranks 32, batch 256: 72.9 -> 66.7 us)
    static constexpr int DEPTH = DEEP && !RUNS && MB1 <= 2 ? 3 : RUNS && !DEEP ? 1 : 2;         // steps in registers: the one being multiplied and those on their way
    const TdcChain3Args &a;
    tdc_rsrc xrs, urs;
    int lane, g, l16, wave, h0, w0, wa, n_units;
    int fu, fs, fmg;                                   // fetch cursor: unit, step, channel group of the unit
    unsigned xoff[PB], woff[MB1];           // byte offsets of the unit's pixels (channel 4g) and weights, or out of range
    float x_top[PB];                                   // largest magnitude of x at this lane's pixels so far
    unsigned smallest = ~0u, smallest_x = ~0u;         // of the pixels' largest sums and of their largest x the smallest (tdc_smallest)
    int x_exp = 0;                                     // x is multiplied by 2^x_exp

    __device__ __forceinline__ Chain3Stage1(const TdcChain3Args &args, int lane_, int wave_, int b, int h0_, int w0_) : a(args)
    {
        lane = lane_; g = lane >> 4; l16 = lane & 15; wave = wave_; h0 = h0_; w0 = w0_;
        wa = w0 > 0 ? (w0 & ~3) : 0;
        const int HW = a.H * a.W;
        xrs = tdc_make_rsrc(a.x + (size_t)b * a.C * HW, (unsigned)a.C * HW * 4u);
        urs = tdc_make_rsrc(a.uin, a.uin_bytes);
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
            xoff[pb] = (ok ? (unsigned)(h * a.W + w) * (NHWC ? 4u * a.C : 4u) : TDC_OOB) + (NHWC ? 16u * g : 16u * g * (unsigned)(a.H * a.W));
        }
#pragma unroll
        for (int mb = 0; mb < MB1; ++mb) {
            const int blk = fmg * MB1 + mb;
            woff[mb] = live && blk < a.NB1 ? (unsigned)(blk * a.S1) * (1024u * NP) + lane * 16u : TDC_OOB;
        }
    }
    __device__ __forceinline__ static tdc_f4 load4(tdc_rsrc r, unsigned off, unsigned soff)
    {
        return __builtin_bit_cast(tdc_f4, (tdc_u4)__builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)soff, 0));
    }
    __device__ __forceinline__ static float load1(tdc_rsrc r, unsigned off, unsigned soff)
    {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, (int)soff, 0));
    }
    // Except in runs a step moves the scalar offset alone; where a last step goes past C, its lanes' offsets are checked one by
    // one.  (NCHW channels past C lie beyond the descriptor by themselves, but only per-lane offsets are certain to be compared with it.)
    __device__ __forceinline__ void fetch(tdc_f4 (&x)[NR], tdc_op<NP> (&w)[MB1])
    {
        const unsigned HW4 = (unsigned)(a.H * a.W) * 4u;
        if (RUNS) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) x[4 * h + j] = load4(xrs, ((unsigned)(32 * fs + 16 * h + j) * HW4 + xoff[0]) | (xoff[0] & TDC_OOB), 0);
        } else if (32 * fs + 32 <= a.C) {
            const unsigned s = (NHWC ? 128u : 32u * HW4) * fs;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    tdc_f4 &v = x[(2 * pb + h) % NR];
                    if (NHWC) v = load4(xrs, xoff[pb] + 64u * h, s);
                    else v = (tdc_f4){load1(xrs, xoff[pb], s + 16 * h * HW4), load1(xrs, xoff[pb], s + (16 * h + 1) * HW4),
                                      load1(xrs, xoff[pb], s + (16 * h + 2) * HW4), load1(xrs, xoff[pb], s + (16 * h + 3) * HW4)};
                }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c = 32 * fs + 16 * h;                  // the lane's are c + 4g ..
                const auto past = [&](int j) { return c + 4 * g + j < a.C ? 0u : TDC_OOB; };
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    tdc_f4 &v = x[(2 * pb + h) % NR];
                    if (NHWC) {
                        v = load4(xrs, (xoff[pb] + 4u * c) | past(0) | (xoff[pb] & TDC_OOB), 0);
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) v[j] = load1(xrs, ((unsigned)(c + j) * HW4 + xoff[pb]) | past(j) | (xoff[pb] & TDC_OOB), 0);
                    }
                }
            }
        }
#pragma unroll
        for (int mb = 0; mb < MB1; ++mb)
#pragma unroll
            for (int q = 0; q < NP; ++q) w[mb].p[q] = __builtin_bit_cast(tdc_h8, load4(urs, woff[mb] + q * 1024u, fs * (1024u * NP)));
        if (++fs == a.S1) {
            fu += TDC_CHAIN3_WAVES;
            place();
        }
    }
    // tile cells whose image column is outside [0, W): the runs never produce them
    __device__ __forceinline__ void zero_outside(tdc_u2 *__restrict__ z1s) const
    {
        if (!RUNS) return;
        const int left = max(-w0, 0), right = max(w0 + a.QW - a.W, 0);
        const int per_row = left + right, total = per_row * a.QH * 4 * NP * a.NB1;
        for (int e = 64 * wave + lane; e < total; e += 64 * TDC_CHAIN3_WAVES) {
            const int c = e % per_row, r = (e / per_row) % a.QH, pl = e / (per_row * a.QH);
            const int qw = c < left ? c : a.QW - right + (c - left);
            z1s[pl * a.pitch1 + r * a.QW + qw] = (tdc_u2){0u, 0u};
        }
    }
    __device__ __forceinline__ void multiply(tdc_f4 (&acc)[MB1][PB][TDC_LEVELS], const tdc_f4 (&x)[NR], const tdc_op<NP> (&w)[MB1])
    {
        const TdcScale s(x_exp);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            const tdc_f4 lo = RUNS ? (tdc_f4){x[0][pb], x[1][pb], x[2][pb], x[3][pb]} : x[(2 * pb) % NR];
            const tdc_f4 hi = RUNS ? (tdc_f4){x[4 % NR][pb], x[5 % NR][pb], x[6 % NR][pb], x[7 % NR][pb]} : x[(2 * pb + 1) % NR];
            x_top[pb] = tdc_largest(tdc_largest(x_top[pb], lo), hi);
            const tdc_op<NP> b = tdc_split_op<NP>(lo, hi, s);
#pragma unroll
            for (int i = 0; i < TdcProducts<NP>::N; ++i)
#pragma unroll
                for (int mb = 0; mb < MB1; ++mb) {
                    tdc_f4 &c = acc[mb][pb][TdcProducts<NP>::level[i]];
                    c = tdc_mfma_part<NP>(i, w[mb].p, b.p, c);
                }
        }
    }
    // the sums of a unit, from their levels, as parts of z1
    __device__ __forceinline__ void store(tdc_u2 *__restrict__ z1s, int unit, const tdc_f4 (&acc)[MB1][PB][TDC_LEVELS])
    {
        const int pg = tdc_div(unit, a.div_mg1), mg = unit - pg * a.n_mg1;
        const int rho = 16 * pg + l16, qh = RUNS ? tdc_div(rho, a.div_RPR) : 0;
        const int qw0 = RUNS ? wa + 4 * (rho - qh * a.RPR) - w0 : 0;
        const TdcScale s(-a.z1_exp);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            const bool ok = RUNS ? qh < a.QH && qw0 + pb >= 0 && qw0 + pb < a.QW : pg * PB + pb < a.QB;
            const int pix = RUNS ? qh * a.QW + qw0 + pb : 16 * (pg * PB + pb) + l16;
            float m = 0.f;
#pragma unroll
            for (int mb = 0; mb < MB1; ++mb) {
                const int blk = mg * MB1 + mb;
                const tdc_f4 v = tdc_levels(acc[mb][pb]);
                m = tdc_largest(m, v);
                tdc_u2 p[NP];
                tdc_split4<NP>(v, s, p);
                if (ok && blk < a.NB1) {
#pragma unroll
                    for (int q = 0; q < NP; ++q) z1s[((q * a.NB1 + blk) * 4 + g) * a.pitch1 + pix] = p[q];
                }
            }
            smallest = tdc_smallest(smallest, tdc_pixel_max(m));
            smallest_x = tdc_smallest(smallest_x, tdc_pixel_max(x_top[pb]));
        }
    }
    __device__ __forceinline__ void run(Chain3Shared &sh, tdc_u2 *__restrict__ z1s)
    {
        tdc_f4 x[DEPTH][NR], acc[MB1][PB][TDC_LEVELS];
        tdc_op<NP> w[DEPTH][MB1];
#pragma unroll
        for (int i = 0; i == 0 || i + 1 < DEPTH; ++i) fetch(x[i], w[i]);
        zero_outside(z1s);
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < NR; ++i) m = tdc_largest_number(m, x[0][i]);
        sh.first[wave] = tdc_wave_max(m);
        __syncthreads();
        x_exp = chain3_x_exp(sh);
        const int total = wave < n_units ? (n_units - wave + TDC_CHAIN3_WAVES - 1) / TDC_CHAIN3_WAVES * a.S1 : 0;
        int unit = wave, step = 0;
        const auto clear = [&]() {
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) x_top[pb] = 0.f;
#pragma unroll
            for (int mb = 0; mb < MB1; ++mb)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int q = 0; q < TDC_LEVELS; ++q) acc[mb][pb][q] = tdc_f4_zero();
        };
        const auto done = [&]() {
            if (++step < a.S1) return;
            store(z1s, unit, acc);
            unit += TDC_CHAIN3_WAVES;
            step = 0;
            clear();
        };
        clear();
        for (int i = 0; i < total; i += DEPTH) {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                if (i + u >= total) break;
                if (DEPTH > 1) fetch(x[(u + DEPTH - 1) % DEPTH], w[(u + DEPTH - 1) % DEPTH]);
                multiply(acc, x[u], w[u]);
                if (DEPTH == 1) fetch(x[0], w[0]);
                done();
            }
        }
    }
};

// The image and the tile of this workgroup: one contiguous range of (image, tile) pairs per XCD, so that halos are shared
// within its L2.
struct Chain3Tile {
    int b, i0, j0;
    __device__ __forceinline__ Chain3Tile(const TdcChain3Args &a)
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
__device__ __forceinline__ void chain3_z1_base(const TdcChain3Args &a, int group, int lane, int (&qbase)[PB])
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
struct Chain3Out {
    const TdcChain3Args &a;
    int g, l16, b, P2;
    tdc_rsrc yrs;
    unsigned yq[PB][4];      // NCHW: byte offset of pixel 4*g + i of block pb in one channel plane, or TDC_OOB
    int ypix[PB];            // NHWC: index of pixel l16 of block pb in the output image, or -1

    __device__ __forceinline__ Chain3Out(const TdcChain3Args &args, const Chain3Tile &at, int group, int lane) : a(args)
    {
        g = lane >> 4; l16 = lane & 15; b = at.b;
        P2 = a.Ho * a.Wo;
        yrs = tdc_make_rsrc(a.y + (size_t)b * a.N * P2, (unsigned)a.N * P2 * 4u);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            const int p0 = 16 * (group * PB + pb) + (NHWC ? l16 : 4 * g);
            const int ph = tdc_div(p0, a.div_TW);
            int pw = p0 - ph * a.TW, oi = at.i0 + ph;
            if (NHWC) {
                const int oj = at.j0 + pw;
                ypix[pb] = (p0 < a.P && oi < a.Ho && oj < a.Wo) ? oi * a.Wo + oj : -1;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (i && ++pw == a.TW) {
                        pw = 0;
                        ++oi;
                    }
                    yq[pb][i] = (p0 + i < a.P && oi < a.Ho && at.j0 + pw < a.Wo) ? (unsigned)(oi * a.Wo + at.j0 + pw) * 4u : TDC_OOB;
                }
            }
        }
    }
    // What the epilogue reads for a lane's outputs of one block.  NCHW rows that allow no quads read their shortcut one by one,
    // where it is added.
    struct Epi {
        float bias[NHWC ? 4 : 1];
        tdc_f4 residual[PB];
    };
    __device__ __forceinline__ void fetch_epi(int nb, Epi &e) const
    {
        const int n = 16 * nb + (NHWC ? 4 * g : l16);
        const bool live = n < a.N;
#pragma unroll
        for (int i = 0; i < (NHWC ? 4 : 1); ++i) e.bias[i] = a.epi.bias && live ? a.epi.bias[n + i] : 0.f;
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            const bool ok = live && (NHWC ? ypix[pb] >= 0 : a.vec && !(yq[pb][0] & TDC_OOB));
            const size_t cell = NHWC ? ((size_t)b * P2 + ypix[pb]) * a.N + n : ((size_t)b * a.N + n) * P2 + (yq[pb][0] >> 2);
            e.residual[pb] = a.epi.residual && ok ? *reinterpret_cast<const tdc_f4 *>(a.epi.residual + cell) : tdc_f4_zero();
        }
    }
    // sums of output block nb, through the epilogue; `e`: fetched before, or null
    template <bool EPI>
    __device__ __forceinline__ void put(int nb, tdc_f4 (&acc3)[PB], const Epi *e) const
    {
        if constexpr (EPI) {
            Epi here;
            if (!e) {
                fetch_epi(nb, here);
                e = &here;
            }
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
#pragma unroll
                for (int i = 0; i < 4; ++i) acc3[pb][i] += e->bias[NHWC ? i : 0];
                if (a.epi.residual) acc3[pb] += e->residual[pb];
            }
            if (!NHWC && !a.vec && a.epi.residual) {
                const int n = 16 * nb + l16;
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (n < a.N && !(yq[pb][i] & TDC_OOB)) acc3[pb][i] += a.epi.residual[((size_t)b * a.N + n) * P2 + (yq[pb][i] >> 2)];
            }
            if (a.epi.relu) {
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc3[pb][i] = fmaxf(acc3[pb][i], 0.f);
            }
        }
        if (NHWC) {
            const int n = 16 * nb + 4 * g;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
                if (ypix[pb] >= 0 && n < a.N) tdc_store4_stream(reinterpret_cast<tdc_f4 *>(a.y + ((size_t)b * P2 + ypix[pb]) * a.N + n), acc3[pb]);
            return;
        }
        // channels past N lie beyond the descriptor: the hardware drops those stores
        const unsigned row = (unsigned)(16 * nb + l16) * P2 * 4u;
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

// Whether the NaNs among a tile's outputs are x's: there is one, all weights are numbers and in parts, and nothing that is no NaN overflowed
// in x or z1.  The outputs then are what fp32 gives.  For the workgroup.
template <int LAY>
__device__ __forceinline__ bool chain3_nan_explained(const TdcChain3Args &a, Chain3Shared &sh, const tdc_u2 *__restrict__ z1s, int lane, int wave)
{
    constexpr bool NHWC = LAY == TDC_LAY_NHWC;
    if (*reinterpret_cast<const int *>(static_cast<const char *>(a.uin) + a.uin_bytes)) return false;
    const int g = lane >> 4, l16 = lane & 15;
    const Chain3Tile at(a);
    const int HW = a.H * a.W;
    const tdc_rsrc xrs = tdc_make_rsrc(a.x + (size_t)at.b * a.C * HW, (unsigned)a.C * HW * 4u);
    TdcFactors xs;
#pragma unroll 1
    for (int qb = wave; qb < a.QB; qb += TDC_CHAIN3_WAVES) {
        const int q = 16 * qb + l16, qh = tdc_div(q, a.div_QW);
        const int h = at.i0 * a.stride - a.pad + qh, w = at.j0 * a.stride - a.pad + q - qh * a.QW;
        const bool in = q < a.Q && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
        const int pix = in ? h * a.W + w : 0;
#pragma unroll 4
        for (int kc = 0; kc < a.C; kc += 16) {
            const int c = kc + 4 * g;
            tdc_f4 x;
            if (NHWC) {
                x = tdc_buf_load4(xrs, in && c < a.C ? (unsigned)(pix * a.C + c) * 4u : TDC_OOB);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = tdc_buf_load(xrs, in && c + j < a.C ? (unsigned)((c + j) * HW + pix) * 4u : TDC_OOB);
            }
            xs.see(x);
        }
    }
    bool large = ldexpf(xs.largest, chain3_x_exp(sh)) > TDC_FP16_MAX;
#pragma unroll 1
    for (int plane = wave; plane < 4 * a.NB1; plane += TDC_CHAIN3_WAVES)
#pragma unroll 1
        for (int q = lane; q < a.Q; q += 64) {
            const tdc_u2 u = z1s[plane * a.pitch1 + q];          // four first parts: an infinity is a value too large
#pragma unroll
            for (int j = 0; j < 4; ++j) large |= (u[j >> 1] >> 16 * (j & 1) & 0x7fffu) == 0x7c00u;
        }
    __syncthreads();                                             // the scale is read
    sh.first[wave] = (tdc_any_lane(xs.nan) ? CHAIN3_NAN : 0) | (tdc_any_lane(large) ? CHAIN3_TOO_LARGE : 0);
    __syncthreads();
    const tdc_u4 all = *reinterpret_cast<const tdc_u4 *>(sh.first);
    return __builtin_amdgcn_readfirstlane((int)(all[0] | all[1] | all[2] | all[3])) == CHAIN3_NAN;
}

// The tile once more in fp32, one load at a time, z1 in fp32 where its parts were (see tdc_split.h).
template <int NB2, int PB, int LAY>
__device__ __forceinline__ void chain3_tile_fp32(const TdcChain3Args &a, tdc_u2 *__restrict__ z1s, int lane, int wave)
{
    constexpr bool NHWC = LAY == TDC_LAY_NHWC;
    tdc_f4 *__restrict__ z1f = reinterpret_cast<tdc_f4 *>(z1s);
    const int g = lane >> 4, l16 = lane & 15;
    const Chain3Tile at(a);
    const int HW = a.H * a.W, KG1 = (a.C + 15) / 16;
    const tdc_rsrc urs = tdc_make_rsrc(tdc_raw_base(a.uin, a.uin_bytes, a.NB1), 1024u * a.NB1 * KG1);
    const tdc_rsrc crs = tdc_make_rsrc(tdc_raw_base(a.core, a.core_bytes, NB2), 1024u * NB2 * a.KG2);
    const tdc_rsrc ors = tdc_make_rsrc(tdc_raw_base(a.uout, a.uout_bytes, a.NB3), 1024u * a.NB3 * NB2);
    const tdc_rsrc xrs = tdc_make_rsrc(a.x + (size_t)at.b * a.C * HW, (unsigned)a.C * HW * 4u);
#pragma unroll 1
    for (int qb = wave; qb < a.QB; qb += TDC_CHAIN3_WAVES) {
        const int q = 16 * qb + l16, qh = tdc_div(q, a.div_QW);
        const int h = at.i0 * a.stride - a.pad + qh, w = at.j0 * a.stride - a.pad + q - qh * a.QW;
        const bool in = q < a.Q && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
        const int pix = in ? h * a.W + w : 0;
#pragma unroll 1
        for (int blk = 0; blk < a.NB1; ++blk) {
            tdc_f4 acc = tdc_f4_zero();
#pragma unroll 1
            for (int kg = 0; kg < KG1; ++kg) {
                const int c = 16 * kg + 4 * g;
                tdc_f4 x;
                if (NHWC) {
                    x = tdc_buf_load4(xrs, in && c < a.C ? (unsigned)(pix * a.C + c) * 4u : TDC_OOB);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = tdc_buf_load(xrs, in && c + j < a.C ? (unsigned)((c + j) * HW + pix) * 4u : TDC_OOB);
                }
                const tdc_f4 u = tdc_raw_weights(urs, blk, KG1, kg, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j) acc = tdc_mfma(u[j], x[j], acc);
            }
            z1f[(blk * 4 + g) * a.pitch1 + q] = in ? acc : tdc_f4_zero();
        }
    }
    __threadfence();         // the outputs stored before are in place, these follow them
    __syncthreads();
    const int slice = wave & ((1 << a.lg_ks) - 1);
#pragma unroll 1
    for (int pg = wave >> a.lg_ks; pg < a.n_pg2; pg += TDC_CHAIN3_WAVES) {
        int qbase[PB];
        chain3_z1_base<PB>(a, pg, lane, qbase);
        tdc_f4 z2[NB2][PB];
#pragma unroll
        for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) z2[mb][pb] = tdc_f4_zero();
#pragma unroll 1
        for (int kg = 0; kg < a.KG2; ++kg) {
            const int tap = tdc_div(kg, a.div_NB1), r = tdc_div(tap, a.div_K), dg = kg - tap * a.NB1;
            const int cell = dg * 4 * a.pitch1 + r * a.QW + tap - r * a.K;
            tdc_f4 z[PB];
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) z[pb] = z1f[cell + qbase[pb]];
#pragma unroll
            for (int mb = 0; mb < NB2; ++mb) {
                const tdc_f4 w = tdc_raw_weights(crs, mb, a.KG2, kg, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb) z2[mb][pb] = tdc_mfma(w[j], z[pb][j], z2[mb][pb]);
            }
        }
        const Chain3Out<PB, NHWC> out(a, at, pg, lane);
#pragma unroll 1
        for (int nb = slice; nb < a.NB3; nb += 1 << a.lg_ks) {
            tdc_f4 acc3[PB];
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) acc3[pb] = tdc_f4_zero();
#pragma unroll
            for (int kg = 0; kg < NB2; ++kg) {
                const tdc_f4 w = tdc_raw_weights(ors, nb, NB2, kg, lane);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb)
                        acc3[pb] = NHWC ? tdc_mfma(w[j], z2[kg][pb][j], acc3[pb]) : tdc_mfma(z2[kg][pb][j], w[j], acc3[pb]);
            }
            out.template put<true>(nb, acc3, nullptr);
        }
    }
}

// Weights that all four wavefronts need, through LDS: chunks of N pieces of 1 KB (a 16-row block's fragment in one part), brought by
// all of them, two chunks ahead in registers, double-buffered.  One fragment then comes through the L1 once per workgroup and
// not once per wavefront: at the 26 to 32 bytes a cycle it delivers, that was the time of stages 2 and 3.
constexpr int chain3_feed_pieces(int nb2)                    // of the larger of the two stages' chunks
{
    const int s3 = (nb2 + 1) / 2, t2 = nb2 == 1 ? 4 : nb2 == 2 ? 2 : 1, u3 = s3 == 1 ? 4 : s3 == 2 ? 2 : 1;
    return NP * (nb2 * t2 > s3 * u3 ? nb2 * t2 : s3 * u3);
}
template <int N>
struct Chain3Feed {
    static constexpr int MINE = (N + TDC_CHAIN3_WAVES - 1) / TDC_CHAIN3_WAVES;
    tdc_f4 r[2][MINE];
    // piece(k): byte offset of piece k of the chunk
    template <class Piece>
    __device__ __forceinline__ void load(int u, tdc_rsrc rs, int lane, int wave, Piece piece)
    {
#pragma unroll
        for (int i = 0; i < MINE; ++i) {
            const int k = wave + TDC_CHAIN3_WAVES * i;
            if (N % TDC_CHAIN3_WAVES == 0 || k < N) r[u][i] = tdc_buf_load4(rs, piece(k) + lane * 16u);
        }
    }
    __device__ __forceinline__ void put(int u, tdc_u4 *__restrict__ buf, int lane, int wave) const
    {
#pragma unroll
        for (int i = 0; i < MINE; ++i) {
            const int k = wave + TDC_CHAIN3_WAVES * i;
            if (N % TDC_CHAIN3_WAVES == 0 || k < N) buf[k * 64 + lane] = __builtin_bit_cast(tdc_u4, r[u][i]);
        }
    }
};

// Not in the deep instances that read NCHW runs: one or two workgroups to a compute unit then wait for HBM in stage 1 and for their
// stores in stage 3, and the barriers cost more than the shared fragments save (128 -> 256 at 56x56 stride 2, batch 32: 26.1
// against 25.4 us; 128 channels at 28x28, ranks 32, batch 256: 72.7 -> 70.5 us).
constexpr bool chain3_shares_weights(int lay, int nb2) { return !(lay == TDC_LAY_NCHW_RUNS && nb2 >= 3); }

// Three and more z2 blocks: the layers whose tiles are large and few, one or two workgroups to a compute unit.  Their instances
// spend the registers on more steps and output blocks on their way instead of on residency.
constexpr bool chain3_deep(int nb2, int pb) { return nb2 >= 3 && pb == 2; }

// Wavefronts per SIMD an instance has registers for; the rarely run code must not cost one.
constexpr int chain3_wavefronts(int nb2, int pb, int lay, int mb1)
{
    if (pb > 2 || nb2 > 2) return 2;
    return lay == TDC_LAY_NCHW_RUNS ? (mb1 <= 2 ? 3 : 2) : lay == TDC_LAY_NHWC && mb1 <= 2 ? 4 : 3;
}

// ALL: every wavefront has a group of pixel blocks of its own (lg_ks is 0)
template <int NB2, int PB, int LAY, int MB1, bool ALL>
__global__ __launch_bounds__(64 * TDC_CHAIN3_WAVES, chain3_wavefronts(NB2, PB, LAY, MB1)) void tdc_chain3_kernel(TdcChain3Args args)
{
    constexpr bool NHWC = LAY == TDC_LAY_NHWC, SWAP = !NHWC;
    constexpr bool DEEP = chain3_deep(NB2, PB);
    extern __shared__ tdc_u4 chain3_lds[];                       // Chain3Shared, z1 [NP parts][NB1][4][pitch1], the partial sums of ks > 1
    Chain3Shared &sh = *reinterpret_cast<Chain3Shared *>(chain3_lds);
    tdc_u2 *__restrict__ z1s = reinterpret_cast<tdc_u2 *>(chain3_lds + sizeof(Chain3Shared) / 16);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bool bad;                                                    // a pixel of too small factors, or a channel of too small outputs
    bool no_number = false;                                      // an output
    int x_exp;
    const Chain3Tile at(args);
    {
        Chain3Stage1<LAY, MB1, DEEP> s1(args, lane, wave, at.b, at.i0 * args.stride - args.pad, at.j0 * args.stride - args.pad);
        s1.run(sh, z1s);
        x_exp = s1.x_exp;
        bad = tdc_is_small(s1.smallest, tdc_exp2i(args.z1_exp + TDC_LOWEST)) || tdc_is_small(s1.smallest_x, tdc_exp2i(max(TDC_LOWEST - x_exp, -126)));
    }

    const TdcChain3Args a = tdc_args_again<TdcChain3Args>();    // read anew, and not kept through stage 1
    const int plane = a.NB1 * 4 * a.pitch1;                      // cells of one part
    const tdc_rsrc crs = tdc_make_rsrc(a.core, a.core_bytes + 64u * NB2), ors = tdc_make_rsrc(a.uout, a.uout_bytes + 64u * a.NB3);   // with the exponents
    // with fewer groups than wavefronts 2 or 4 of them share one: each takes a slice of stage 2's contraction, the sums meet in
    // LDS, and each takes every ks-th output block of stage 3 (the loop then runs once for every wavefront).  Else every
    // wavefront has a group, all need the same weights, and share them.
    const int lg_ks = ALL ? 0 : a.lg_ks, ks = 1 << lg_ks, slice = wave & (ks - 1);
    constexpr int S3 = (NB2 + 1) / 2;
    constexpr int T2 = NB2 == 1 ? 4 : NB2 == 2 ? 2 : 1, U3 = S3 == 1 ? 4 : S3 == 2 ? 2 : 1;    // steps, output blocks of a chunk
    constexpr int PIECES = chain3_feed_pieces(NB2);
    tdc_u4 *__restrict__ feed = reinterpret_cast<tdc_u4 *>(z1s + NP * plane);                  // two chunks
    for (int round = 0; round < a.n_pg2; round += TDC_CHAIN3_WAVES >> lg_ks) {
        const int pg = round + (wave >> lg_ks);
        const bool live = pg < a.n_pg2;
        // ---- stage 2: z2 channels 16*mb + 4*g + {0..3} of pixel l16 of block pb
        int qbase[PB];
        chain3_z1_base<PB>(a, pg, lane, qbase);
        tdc_f4 z2[NB2][PB];
        {
            tdc_f4 acc2[NB2][PB][TDC_LEVELS];
#pragma unroll
            for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int q = 0; q < TDC_LEVELS; ++q) acc2[mb][pb][q] = tdc_f4_zero();
            // a fetch past the last step stays inside the descriptor or reads 0, and is never multiplied
            const auto fetch_w = [&](int step, tdc_op<NP>(&w)[NB2]) {
#pragma unroll
                for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
                    for (int q = 0; q < NP; ++q)
                        w[mb].p[q] = __builtin_bit_cast(tdc_h8, tdc_buf_load4(crs, ((unsigned)(mb * a.S2 + step) * NP + q) * 1024u + lane * 16u));
            };
            const int st0 = slice * a.S2 >> lg_ks, st1 = (slice + 1) * a.S2 >> lg_ks;
            // cell of the next k-group: channel block dg of tap (r, s)
            int kg = 2 * st0;
            const int tap = tdc_div(kg, a.div_NB1), r = tdc_div(tap, a.div_K), step_dg = 4 * a.pitch1, step_tap = 1 - a.NB1 * step_dg, step_row = a.QW - a.K;
            int dg = kg - tap * a.NB1, s = tap - r * a.K, cell = dg * step_dg + r * a.QW + s;
            const auto next_cell = [&]() {
                const int here = cell;
                ++kg;
                cell += step_dg;
                if (++dg == a.NB1) {
                    dg = 0;
                    cell += step_tap;
                    if (++s == a.K) {
                        s = 0;
                        cell += step_row;
                    }
                }
                return here;
            };
            // z1 of the next step, one ahead of its products; past the last one any cell does
            const auto read_z1 = [&](tdc_op<NP>(&o)[PB]) {
                int lo = next_cell();
                lo = kg <= a.KG2 ? lo : 0;
                const bool whole = kg < a.KG2;                   // else the last half step, whose weights are zero: any finite cell does
                const int nx = next_cell(), hi = whole ? nx : lo;
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int q = 0; q < NP; ++q) {
                        const tdc_u2 u = z1s[q * plane + lo + qbase[pb]], v = z1s[q * plane + hi + qbase[pb]];
                        o[pb].p[q] = __builtin_bit_cast(tdc_h8, (tdc_u4){u[0], u[1], v[0], v[1]});
                    }
            };
            const auto step2 = [&](const tdc_op<NP>(&w)[NB2], const tdc_op<NP>(&z)[PB]) {
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int i = 0; i < TdcProducts<NP>::N; ++i)
#pragma unroll
                        for (int mb = 0; mb < NB2; ++mb) {
                            tdc_f4 &c = acc2[mb][pb][TdcProducts<NP>::level[i]];
                            c = tdc_mfma_part<NP>(i, w[mb].p, z[pb].p, c);
                        }
            };
            tdc_op<NP> z[2][PB];
            if constexpr (ALL) {
                Chain3Feed<NB2 * T2 * NP> f;
                const auto load = [&](int u, int chunk) {
                    f.load(u, crs, lane, wave, [&](int k) {
                        const int mb = k / (T2 * NP);
                        return (unsigned)((mb * a.S2 + chunk * T2) * NP + k - mb * T2 * NP) * 1024u;
                    });
                };
                load(0, 0);
                load(1, 1);
                __syncthreads();                                 // z1 is there, or the chunks of the last round are read
                f.put(0, feed, lane, wave);
                const int chunks = (a.S2 + T2 - 1) / T2;
                const auto read_w = [&](int u, int t, tdc_op<NP>(&w)[NB2]) {
#pragma unroll
                    for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
                        for (int q = 0; q < NP; ++q) w[mb].p[q] = __builtin_bit_cast(tdc_h8, feed[(u * PIECES + (mb * T2 + t) * NP + q) * 64 + lane]);
                };
                read_z1(z[0]);
                for (int c = 0; c < chunks; c += 2) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        if (c + u >= chunks) break;
                        __syncthreads();
                        load(u, c + u + 2);
#pragma unroll
                        for (int t = 0; t < T2; ++t) {
                            if (!live || (c + u) * T2 + t >= a.S2) break;
                            tdc_op<NP> w[NB2];
                            read_w(u, t, w);
                            const int i = T2 == 1 ? u : t & 1;
                            read_z1(z[1 - i]);
                            step2(w, z[i]);
                        }
                        f.put(1 - u, feed + (1 - u) * PIECES * 64, lane, wave);
                    }
                }
            } else {
                constexpr int DEPTH = 2;
                tdc_op<NP> w[DEPTH][NB2];
#pragma unroll
                for (int i = 0; i + 1 < DEPTH; ++i) fetch_w(st0 + i, w[i]);
                __syncthreads();                                 // z1 is there
                read_z1(z[0]);
                for (int st = st0; st < st1; st += DEPTH) {
#pragma unroll
                    for (int u = 0; u < DEPTH; ++u) {
                        if (st + u >= st1) break;
                        fetch_w(st + u + DEPTH - 1, w[(u + DEPTH - 1) % DEPTH]);
                        read_z1(z[1 - u]);
                        step2(w[u], z[u]);
                    }
                }
            }
            // to a common scale
#pragma unroll
            for (int mb = 0; mb < NB2; ++mb) {
                const tdc_u4 e = __builtin_bit_cast(tdc_u4, tdc_buf_load4(crs, a.core_bytes + (16u * mb + 4u * (lane >> 4)) * 4u));
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    z2[mb][pb] = tdc_levels(acc2[mb][pb]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) z2[mb][pb][i] = ldexpf(z2[mb][pb][i], (int)e[i]);
                }
            }
        }
        if (ks > 1) {      // partial sums, added in the order of the slices
            tdc_f4 *__restrict__ red = reinterpret_cast<tdc_f4 *>(z1s + NP * plane);
#pragma unroll
            for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) red[((wave * NB2 + mb) * PB + pb) * 64 + lane] = z2[mb][pb];
            __syncthreads();
            const int first = wave - slice;
#pragma unroll
            for (int mb = 0; mb < NB2; ++mb)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    tdc_f4 v = red[((first * NB2 + mb) * PB + pb) * 64 + lane];
                    for (int j = 1; j < ks; ++j) v += red[(((first + j) * NB2 + mb) * PB + pb) * 64 + lane];
                    z2[mb][pb] = v;
                }
        }
        // ---- stage 3, operands swapped in NCHW: D[pixel 4*g + i][channel l16]; NHWC: D[channel 4*g + i][pixel l16]
        struct Exponents {
            int e[NHWC ? 4 : 1];                                 // of the lane's output channels
        };
        const auto fetch_e = [&](int nb, Exponents &u) {
            if constexpr (NHWC) {
                const tdc_u4 e = __builtin_bit_cast(tdc_u4, tdc_buf_load4(ors, a.uout_bytes + (16u * nb + 4u * (lane >> 4)) * 4u));
#pragma unroll
                for (int i = 0; i < 4; ++i) u.e[i] = (int)e[i];
            } else {
                u.e[0] = __builtin_amdgcn_raw_buffer_load_b32(ors, (int)(a.uout_bytes + (16u * nb + (lane & 15)) * 4u), 0, 0);
            }
        };
        const auto fetch = [&](int nb, tdc_op<NP>(&u)[S3]) {
#pragma unroll
            for (int st = 0; st < S3; ++st)
#pragma unroll
                for (int q = 0; q < NP; ++q)
                    u[st].p[q] = __builtin_bit_cast(tdc_h8, tdc_buf_load4(ors, ((unsigned)(nb * S3 + st) * NP + q) * 1024u + lane * 16u));
        };
        // the first weights, under the splitting of z2
        Chain3Feed<U3 * S3 * NP> f3;
        const auto load3 = [&](int u, int chunk) {
            f3.load(u, ors, lane, wave, [&](int k) { return (unsigned)(chunk * U3 * S3 * NP + k) * 1024u; });
        };
        tdc_op<NP> u0[S3], u1[S3];
        if constexpr (ALL) {
            load3(0, 0);
            load3(1, 1);
        } else {
            fetch(slice, u0);
        }
        float top = 0.f;                                         // largest magnitude of z2 that is no NaN
        unsigned smallest = ~0u;                                 // of the pixels' largest z2 values the smallest
        int lit = 0;                                             // pixels at which z2 is not all zero, of those this lane judges (see emit)
        bool first_lit = false;
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            float m = 0.f;
#pragma unroll
            for (int mb = 0; mb < NB2; ++mb) m = tdc_max3_abs(tdc_max3_abs(m, z2[mb][pb][0], z2[mb][pb][1]), z2[mb][pb][2], z2[mb][pb][3]);
            m = tdc_pixel_max(m);
            top = __builtin_elementwise_maximum(top, m);
            smallest = tdc_smallest(smallest, m);
            const int p = 16 * (pg * PB + pb) + (lane & 15);
            lit += NHWC ? m != 0.f && p < a.P : __builtin_popcount((unsigned)__builtin_amdgcn_ballot_w64(m != 0.f && p < a.P) >> 4 * (lane >> 4) & 15u);
            first_lit |= m != 0.f && p >= a.P;                   // past the last pixel the first stands in
        }
        if (NHWC) {
            lit += tdc_row_ror8(lit);
            lit += (int)(lit > 0) & (int)((first_lit | tdc_row_ror8(first_lit)) != 0) & (int)(pg * PB * 16 + (lane & 7) != 0);
        }
        // Few sums may be small by chance, four hardly ever: lanes of fewer are judged only where a wavefront has no others.  (128 -> 128 at
        // 28x28, batch 10, NHWC, tiles of 5 x 7, whose last blocks hold three pixels: judged by lanes of one or two pixels each, three
        // of four layers of a network ran a tile twice, 30 us instead of 12.)
        const bool judged = lit > (tdc_any_lane(lit > 3) ? 3 : tdc_any_lane(lit > 1) ? 1 : 0);
        const int z2_exp = tdc_scale_of(tdc_wave_max(top), TDC_Z2_TARGET, 0);
        bad |= tdc_is_small(smallest, tdc_exp2i(max(TDC_LOWEST - z2_exp, -126)));
        const int y_exp = a.z1_exp - z2_exp - x_exp;            // y is 2^(y_exp - exponent of the channel) times its sum
        tdc_op<NP> zb[S3][PB];
        {
            const TdcScale s(z2_exp);
#pragma unroll
            for (int st = 0; st < S3; ++st)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
                    zb[st][pb] = tdc_split_op<NP>(z2[2 * st][pb], 2 * st + 1 < NB2 ? z2[(2 * st + 1) % NB2][pb] : tdc_f4_zero(), s);
        }
        const Chain3Out<PB, NHWC> out(a, at, pg, lane);
        float largest = 0.f;
        const int lost = judged ? (127 + min(max(z2_exp + a.lost2, a.lost3), 126)) << 23 : 0;
        int least = 0x7f800000;                                  // of the magnitudes of the channels' largest sums the least, as bits
        // two instances of the loop, as in tdc_chain_kernel.h: without epilogue loads nothing ever waits for the stores
        typedef typename Chain3Out<PB, NHWC>::Epi Epi;
        const auto emit = [&](auto with_epi, int nb, const tdc_op<NP>(&u)[S3], const Exponents &e, const Epi *epi) {
            tdc_f4 acc3[PB][TDC_LEVELS], v[PB];
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int q = 0; q < TDC_LEVELS; ++q) acc3[pb][q] = tdc_f4_zero();
#pragma unroll
            for (int st = 0; st < S3; ++st)
#pragma unroll
                for (int i = 0; i < TdcProducts<NP>::N; ++i)
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb) {
                        tdc_f4 &c = acc3[pb][TdcProducts<NP>::level[i]];
                        c = tdc_mfma_part<NP, SWAP>(i, u[st].p, zb[st][pb].p, c);
                    }
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                v[pb] = tdc_levels(acc3[pb]);
                largest = tdc_largest(largest, v[pb]);
            }
            // a channel's largest among this lane's pixels, of those that are no NaN, in NHWC with those of the lane eight further
#pragma unroll
            for (int i = 0; i < (NHWC ? 4 : 1); ++i) {
                float m = fabsf(v[0][i]);
#pragma unroll
                for (int pb = 0; pb < PB; pb += NHWC ? 2 : 1) {
                    if (NHWC) {
                        m = tdc_max3_abs(m, v[pb][i], v[pb + 1][i]);
                    } else {
                        m = tdc_max3_abs(m, v[pb][0], v[pb][1]);
                        m = tdc_max3_abs(m, v[pb][2], v[pb][3]);
                    }
                }
                const int bits = __builtin_bit_cast(int, m);
                least = min(least, NHWC ? max(bits, tdc_row_ror8(bits)) : bits);
            }
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[pb][i] = ldexpf(v[pb][i], y_exp - e.e[NHWC ? i : 0]);
            out.template put<decltype(with_epi)::value>(nb, v, epi);
        };
        const auto stage3 = [&](auto with_epi) {
            // exponents, and in the deep instances bias and shortcut, one block ahead
            constexpr bool AHEAD = DEEP && decltype(with_epi)::value;
            Exponents ex[2];
            Epi epi[2];
            const auto ahead = [&](int nb, int i) {
                fetch_e(nb, ex[i]);
                if constexpr (AHEAD) out.fetch_epi(nb, epi[i]);
            };
            ahead(slice, 0);
            if constexpr (ALL) {
                __syncthreads();                                 // stage 2 has read its chunks
                f3.put(0, feed, lane, wave);
                const int chunks = (a.NB3 + U3 - 1) / U3;
                for (int c = 0; c < chunks; c += 2) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if (c + h >= chunks) break;
                        __syncthreads();
                        load3(h, c + h + 2);
#pragma unroll 1
                        for (int j = 0; j < U3; ++j) {
                            const int nb = (c + h) * U3 + j;
                            if (!live || nb >= a.NB3) break;
                            ahead(nb + 1, 1);
                            tdc_op<NP> w[S3];
#pragma unroll
                            for (int st = 0; st < S3; ++st)
#pragma unroll
                                for (int q = 0; q < NP; ++q) w[st].p[q] = __builtin_bit_cast(tdc_h8, feed[(h * PIECES + (j * S3 + st) * NP + q) * 64 + lane]);
                            emit(with_epi, nb, w, ex[0], AHEAD ? &epi[0] : nullptr);
                            ex[0] = ex[1];
                            if constexpr (AHEAD) epi[0] = epi[1];
                        }
                        f3.put(1 - h, feed + (1 - h) * PIECES * 64, lane, wave);
                    }
                }
            } else {
                for (int nb = slice; nb < a.NB3; nb += 2 * ks) {
                    fetch(nb + ks, u1);
                    ahead(nb + ks, 1);
                    emit(with_epi, nb, u0, ex[0], AHEAD ? &epi[0] : nullptr);
                    fetch(nb + 2 * ks, u0);
                    ahead(nb + 2 * ks, 0);
                    if (nb + ks < a.NB3) emit(with_epi, nb + ks, u1, ex[1], AHEAD ? &epi[1] : nullptr);
                }
            }
        };
        if (a.epi.bias || a.epi.residual || a.epi.relu) stage3(std::true_type{});
        else stage3(std::false_type{});
        bad |= least < lost;
        no_number |= !tdc_finite(largest);
    }
    // One wavefront's trouble is the tile's: z1 is everybody's.
    sh.bad[wave] = (tdc_any_lane(bad) ? CHAIN3_SMALL : 0) | (tdc_any_lane(no_number) ? CHAIN3_NO_NUMBER : 0);
    __syncthreads();
    const tdc_u4 all = *reinterpret_cast<const tdc_u4 *>(sh.bad);
    const unsigned any = (unsigned)__builtin_amdgcn_readfirstlane((int)(all[0] | all[1] | all[2] | all[3]));
    if (__builtin_expect(any, 0)) {
        const TdcChain3Args &cold = tdc_args_again<TdcChain3Args>();
        if (any == CHAIN3_NO_NUMBER && chain3_nan_explained<LAY>(cold, sh, z1s, lane, wave)) return;
        chain3_tile_fp32<NB2, PB, LAY>(cold, z1s, lane, wave);
    }
}

}  // namespace

// (z2 blocks, pixel blocks of a unit) that have an instance: what fits 256 registers beside the weights in flight, or nearly
// so (three z2 blocks with PB = 4 in NCHW)
#define TDC_CHAIN3_UNITS(X) X(1, 4) X(2, 4) X(3, 4) X(1, 2) X(2, 2) X(3, 2) X(4, 2) X(5, 2)

template <int LAY>
hipError_t tdc_launch_chain3_lay(const TdcChain3Args &a, int nb2, int pb, int mb1, dim3 grid, size_t lds, hipStream_t s, bool prepare_only)
{
#define TDC_LAUNCH(N_, P_, M_, ALL_)                                                                              \
    if (mb1 == M_ && (chain3_shares_weights(LAY, N_) && a.lg_ks == 0) == ALL_) {                                                         \
        hipError_t e = tdc_allow_lds((const void *)tdc_chain3_kernel<N_, P_, LAY, M_, ALL_>, lds);                 \
        if (e != hipSuccess || prepare_only) return e;                                                                 \
        hipLaunchKernelGGL((tdc_chain3_kernel<N_, P_, LAY, M_, ALL_>), grid, dim3(64 * TDC_CHAIN3_WAVES), lds, s, a); \
        return hipGetLastError();                                                                                      \
    }
#define TDC_X(N_, P_)                                                                                                  \
    if (nb2 == N_ && pb == P_) {                                                                                       \
        TDC_LAUNCH(N_, P_, 1, true) TDC_LAUNCH(N_, P_, 2, true) TDC_LAUNCH(N_, P_, 3, true)                            \
        TDC_LAUNCH(N_, P_, 1, false) TDC_LAUNCH(N_, P_, 2, false) TDC_LAUNCH(N_, P_, 3, false)                      \
    }
    TDC_CHAIN3_UNITS(TDC_X)
#undef TDC_X
#undef TDC_LAUNCH
    return hipErrorInvalidValue;
}

#endif
