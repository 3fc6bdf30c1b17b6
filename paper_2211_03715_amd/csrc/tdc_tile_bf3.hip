// The dense layer for launches that are bound by matrix arithmetic or by memory bandwidth, not by latency: an implicit GEMM
//   D[m][p] = sum_k Wt[k][m] * Act[k][p]
// in TM x 64 tiles (output channels x pixels), fp32 in and out, products in three bf16 parts (tdc_bf3.h).
// For contractions of at most 72 terms (tdc_tile_bf3), where two fp16 parts (tdc_tile.hip) are the less accurate form and the first look at
// x that three of them need is not hidden; the figures of longer contractions below are from before those went to two fp16 parts.
//
// Pixels are numbered through the whole batch, p = b*P + (pixel of image b), so small images leave no part-empty tiles.
// A workgroup is KS groups of four wavefronts; the contraction goes in steps of two 16-wide k-groups (tap, channel block),
// dealt to the groups in turn.  The activations of a step are brought in by all threads of a group, fp32 from memory (two
// steps ahead, in registers), split into their parts once and handed to the group's wavefronts through LDS, double-buffered:
// one barrier per step.  The weights were split when they were re-laid out; a wavefront loads its own fragments straight
// into registers, one step ahead.
//
// What bounds it, and why this form.  The six products per fp32 product cost 768 cycles of the matrix cores for a
// 128 x 64 step.  The other resources of a compute unit are then all about half busy: the L1 path (54 bytes a cycle
// measured; 32 KB a step), LDS (128 bytes a cycle; 60 KB and its conflicts), and instruction issue (an MFMA leaves room for
// two other vector instructions: the conversions are placed between them).  Measured variants of the loop, 128 x 64, on
// 1024 -> 512 at 14x14, batch 32 (6.6 GFLOP): both operands through LDS, two barriers a step 53 us; no LDS, every wavefront
// loading and splitting its own pixels 64 us (NHWC loads of 16 pixels x 64 bytes run at 18 bytes a cycle, a third of
// contiguous ones); this one without the interleaving 42.8 us, as it stands 39.8 us (fp32 MFMA kernel: 90.5 us).  On large
// products it runs at 209 TFLOP/s of fp32 products, 1250 of bf16 ones -- what the vendor's bf16 GEMM of 8192^3 reaches on
// the card (1241): power, not issue, is the limit there (all-zero operands: 273 TFLOP/s).
#include "tdc_bf3.h"
#include "tdc_internal.h"

namespace {

struct TileArgs {
    const float *act;
    const void *w3;         // weights in three parts, [NBm][S][3][64 lanes][8 bf16] (S steps)
    float *out;
    TdcEpi epi;             // applied where out is the layer's y
    int C;                  // channels of act
    int HW;                 // pixels per image of act
    int M;                  // output channels that exist
    int P, Ptot;            // output pixels per image, in all
    int NBm, NBk, KG, S;    // 16-blocks of M; k-groups per tap; k-groups in all; steps
    int H, W, Wo, K, stride, pad;
    int n_mt, n_pt, pt_major;
    int vec;                // NCHW out: quads of pixels lie in one image and 16-byte aligned
    unsigned w_bytes;
    TdcDiv div_P, div_Wo, div_NBk, div_K, div_inner;
};

__device__ __forceinline__ int tile_logical_block(int bid, int n)
{
    const int per = n / 8, rem = n % 8, xcd = bid % 8, slot = bid / 8;
    return xcd * per + min(xcd, rem) + slot;
}

// One output by fp32 multiply-adds over the taps inside the image.
template <int ACT>
__device__ __forceinline__ void tile_plain_output(const TileArgs &a, int m, int p)
{
    const int b = tdc_div(p, a.div_P), pix = p - b * a.P;
    const int oh = tdc_div(pix, a.div_Wo), h0 = oh * a.stride - a.pad, w0 = (pix - oh * a.Wo) * a.stride - a.pad;
    const float *x = a.act + (size_t)b * a.C * a.HW;
    const unsigned short *w = reinterpret_cast<const unsigned short *>(a.w3) + (size_t)(m >> 4) * a.S * 1536;
    float sum = 0.f;
#pragma unroll 1
    for (int kg = 0; kg < a.KG && sum == sum; ++kg) {
        const int tap = tdc_div(kg, a.div_NBk), c0 = 16 * (kg - tap * a.NBk);
        const int r = tdc_div(tap, a.div_K), h = h0 + r, wx = w0 + tap - r * a.K;
        if (h < 0 || h >= a.H || wx < 0 || wx >= a.W) continue;
        const int q = h * a.W + wx;
#pragma unroll 1
        for (int k = 0; k < 16 && c0 + k < a.C; ++k) {
            const unsigned short *f = w + (size_t)(kg >> 1) * 1536 + ((m & 15) + 16 * (k >> 2)) * 8 + (kg & 1) * 4 + (k & 3);
            sum = fmaf(tdc_join(f[0], f[512], f[1024]), ACT == TDC_ACT_NHWC ? x[(size_t)q * a.C + c0 + k] : x[(size_t)(c0 + k) * a.HW + q], sum);
        }
    }
    const size_t idx = ACT == TDC_ACT_NHWC ? (size_t)p * a.M + m : ((size_t)b * a.M + m) * a.P + pix;
    a.out[idx] = tdc_apply_epilogue(a.epi, sum, m, idx);
}

// A wavefront's sums once more on the fp32 matrix cores, one load at a time (see tdc_bf3.h), unless their NaNs are x's or the
// weights'.  Returns a bit per sum of this lane for those that an infinite weight at a tap outside the image made NaN (it is 0
// times the weight here, and no part of the sum).  3x3, 128 -> 128 at 28x28,
// batch 8, every value NaN: 70 us, 26 with numbers (one output after the other: 5350).
template <int ACT, bool CONV, int MB, int PB>
__device__ __forceinline__ unsigned tile_redo(const TileArgs &a, bool small, int lane, int p_base, int mb0, tdc_f4 (&acc)[MB][PB])
{
    constexpr bool SWAP = ACT == TDC_ACT_NCHW;
    const int g = lane >> 4, l16 = lane & 15;
    const int b0 = tdc_div(p_base, a.div_P), n_img = min((16 * PB - 1) / a.P + 2, tdc_div(a.Ptot - 1, a.div_P) + 1 - b0);
    const size_t img_elems = (size_t)a.C * a.HW;
    const tdc_rsrc ars = tdc_make_rsrc(a.act + (size_t)b0 * img_elems, (unsigned)(n_img * img_elems * 4));
    const tdc_rsrc wrs = tdc_make_rsrc(a.w3, a.w_bytes);
    const auto load_x = [&](int kg, int pb) {      // channels 4*g .. of k-group kg for pixel l16 of block pb; 0 outside
        const int tap = CONV ? tdc_div(kg, a.div_NBk) : 0, c = 16 * (kg - tap * a.NBk) + 4 * g;
        const int r = CONV ? tdc_div(tap, a.div_K) : 0;
        const int p = p_base + 16 * pb + l16;
        const bool ok = p < a.Ptot;
        const int b = tdc_div(ok ? p : p_base, a.div_P), pix = (ok ? p : p_base) - b * a.P;
        const int oh = CONV ? tdc_div(pix, a.div_Wo) : 0;
        const int h = oh * a.stride - a.pad + r, w = (pix - oh * a.Wo) * a.stride - a.pad + tap - r * a.K;
        const bool in = ok && (!CONV || (h >= 0 && h < a.H && w >= 0 && w < a.W));
        const int q = CONV ? h * a.W + w : pix;
        const unsigned o = (unsigned)((b - b0) * (int)img_elems + (ACT == TDC_ACT_NHWC ? q * a.C + c : c * a.HW + q)) * 4u;
        tdc_f4 v;
        if (ACT == TDC_ACT_NHWC) return tdc_buf_load4(ars, in && c < a.C ? o : TDC_OOB);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = tdc_buf_load(ars, in && c + j < a.C ? o + 4u * j * a.HW : TDC_OOB);
        return v;
    };
    const auto load_w = [&](int kg, int mb) { return mb0 + mb < a.NBm ? tdc_join_weights(wrs, mb0 + mb, a.S, kg, lane) : tdc_f4_zero(); };

    TdcFactors xs, ws;
#pragma unroll 2
    for (int kg = 0; kg < a.KG; ++kg) {
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) xs.see(load_x(kg, pb));
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            if (mb0 + mb < a.NBm) ws.see(tdc_first_parts(wrs, mb0 + mb, a.S, kg, lane));
    }
    const bool odd_weights = tdc_any_lane(ws.nan || ws.largest == INFINITY);
    xs.nan |= ws.nan;
    xs.largest = fmaxf(xs.largest, ws.largest);
    if (xs.explain_nan() && !small && !(CONV && odd_weights)) return 0u;

#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc[mb][pb] = tdc_f4_zero();
#pragma unroll 1
    for (int kg = 0; kg < a.KG; ++kg) {
        tdc_f4 x[PB];
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) x[pb] = load_x(kg, pb);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const tdc_f4 w = load_w(kg, mb);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) acc[mb][pb] = SWAP ? tdc_mfma(x[pb][j], w[j], acc[mb][pb]) : tdc_mfma(w[j], x[pb][j], acc[mb][pb]);
        }
    }
    unsigned nans = 0;
    if (CONV && odd_weights) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int i = 0; i < 4; ++i) nans |= acc[mb][pb][i] != acc[mb][pb][i] ? 1u << ((mb * PB + pb) * 4 + i) : 0u;
    }
    return nans;
}

template <int ACT, bool CONV, int WM, int MB, int PB, int KS>
__global__ __launch_bounds__(256 * KS, 3) void tdc_tile_bf3_kernel(TileArgs a)
{
    constexpr int WP = 4 / WM, TM = 16 * MB * WM, TP = 16 * PB * WP;
    constexpr int NX = TP / 32;                    // 16-byte pieces of activations a thread brings per step
    constexpr int PITCH = TP + 4;                  // 16-byte cells
    constexpr int VPM = (NX * (ACT == TDC_ACT_NCHW ? 40 : 34) + 20 + 6 * MB * PB - 1) / (6 * MB * PB);   // VALU instructions per MFMA
    __shared__ tdc_u4 xs_all[KS][2][12 * PITCH];   // [part][lane group][pixel]: 4 channels of each k-group of the step
    const int ks = KS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
    tdc_u4(&xs)[2][12 * PITCH] = xs_all[ks];
    const int t = threadIdx.x & 255, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int g = lane >> 4, l16 = lane & 15;
    const int wm = wave % WM, wp = wave / WM;

    const int lb = tile_logical_block(blockIdx.x, gridDim.x);
    const int inner = a.pt_major ? a.n_mt : a.n_pt;
    const int hi = tdc_div(lb, a.div_inner), lo = lb - hi * inner;
    const int pt = a.pt_major ? hi : lo, mt = a.pt_major ? lo : hi;
    const int p_tile = pt * TP, p_base = p_tile + wp * PB * 16;
    const int mb0 = mt * (TM / 16) + wm * MB;
    const int b0 = tdc_div(p_tile, a.div_P);       // image of the tile's first pixel: offsets are relative to it
    const size_t img_elems = (size_t)a.C * a.HW;
    // the tile's images; the host keeps their span below 2 GiB
    const int n_img = min((TP - 1) / a.P + 2, tdc_div(a.Ptot - 1, a.div_P) + 1 - b0);
    const tdc_rsrc ars = tdc_make_rsrc(a.act + (size_t)b0 * img_elems, (unsigned)(n_img * img_elems * 4));
    const tdc_rsrc wrs = tdc_make_rsrc(a.w3, a.w_bytes);

    // ---- the pixels this thread brings: byte offset of the (0, 0) tap of its first channel, tap position
    constexpr int NPIX = ACT == TDC_ACT_NCHW ? 1 : NX;
    unsigned poff[NPIX];
    int ph[NPIX], pw[NPIX];
    const int c4 = t & 7;                          // NHWC: channels 4*(c4%4).. of k-group c4/4 of the step
    const int nq = t / TP;                         // NCHW: channels 4*(nq*NX/2 + n).. of both k-groups
#pragma unroll
    for (int i = 0; i < NPIX; ++i) {
        const int p = p_tile + (ACT == TDC_ACT_NCHW ? t % TP : (t >> 3) + 32 * i);
        const bool ok = p < a.Ptot;
        const int b = tdc_div(ok ? p : p_tile, a.div_P), pix = (ok ? p : p_tile) - b * a.P;
        int h = 0, w = 0, off = pix;
        if (CONV) {
            const int oh = tdc_div(pix, a.div_Wo);
            h = oh * a.stride - a.pad;
            w = (pix - oh * a.Wo) * a.stride - a.pad;
            off = h * a.W + w;
        }
        ph[i] = ok ? h : -0x10000000;              // a pixel past the end is outside every image
        pw[i] = w;
        const int e = (b - b0) * (int)img_elems + (ACT == TDC_ACT_NHWC ? off * a.C + 4 * c4 : off + 2 * NX * nq * a.HW);
        poff[i] = (unsigned)e * 4u;
        if (!CONV && !ok) poff[i] = TDC_OOB;
    }
    struct KPos {
        int cb, r, s;
    };
    const auto kpos = [&](int kg) {
        KPos k{kg, 0, 0};
        if (CONV) {
            const int tap = tdc_div(kg, a.div_NBk);
            k.cb = kg - tap * a.NBk;
            k.r = tdc_div(tap, a.div_K);
            k.s = tap - k.r * a.K;
        }
        return k;
    };
    // Every "reads nothing" case is the top bit of the offset, taken from the sign of a difference: no branch, so that a step
    // is one basic block whose loads, conversions and MFMAs can be interleaved.
    const auto fetch_x = [&](int step, tdc_f4(&x)[NX]) {
        const unsigned dead = (unsigned)(a.S - 1 - step) & TDC_OOB;      // past the end
        const KPos k0 = kpos(2 * step), k1 = kpos(2 * step + 1);
        const unsigned half = (unsigned)(a.KG - 2 - 2 * step) & TDC_OOB; // the second k-group of the last step may not exist
        if (ACT == TDC_ACT_NHWC) {
            const bool second = c4 & 4;
            const int cb = second ? k1.cb - 1 : k0.cb;      // poff counts 4*c4 channels
            const int r = second ? k1.r : k0.r, s = second ? k1.s : k0.s;
            const unsigned bad = dead | (second ? half : 0u) | ((unsigned)(a.C - 1 - 16 * cb - 4 * c4) & TDC_OOB);
            const unsigned d = (unsigned)((r * a.W + s) * a.C + 16 * cb) * 4u;
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                const unsigned out = CONV ? (unsigned)((ph[i] + r) | (a.H - 1 - ph[i] - r) | (pw[i] + s) | (a.W - 1 - pw[i] - s)) : poff[i];
                x[i] = tdc_buf_load4(ars, (poff[i] + d) | bad | (out & TDC_OOB));
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const KPos k = h ? k1 : k0;
                const int r = k.r, s = k.s;
                const unsigned out = CONV ? (unsigned)((ph[0] + r) | (a.H - 1 - ph[0] - r) | (pw[0] + s) | (a.W - 1 - pw[0] - s)) : poff[0];
                const unsigned o = (poff[0] + (unsigned)(16 * k.cb * a.HW + r * a.W + s) * 4u) | ((out | dead | (h ? half : 0u)) & TDC_OOB);
                const int cleft = a.C - 1 - 16 * k.cb - 2 * NX * nq;     // this thread's last channel that exists
#pragma unroll
                for (int n = 0; n < NX / 2; ++n)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        x[2 * n + h][j] = tdc_buf_load(ars, (o + (unsigned)((4 * n + j) * a.HW) * 4u) | ((o | (unsigned)(cleft - 4 * n - j)) & TDC_OOB));
            }
        }
    };
    // piece i of a step's activations: split and stored as operand halves (NCHW: two pieces, the halves of a cell, at once)
    const auto to_lds = [&](const tdc_f4(&x)[NX], tdc_u4 *__restrict__ xb, int i) {
        if (ACT == TDC_ACT_NHWC) {
            tdc_u2 *__restrict__ x2 = reinterpret_cast<tdc_u2 *>(xb);
            tdc_u2 s[3];
            tdc_split4(x[i], s[0], s[1], s[2]);
#pragma unroll
            for (int q = 0; q < 3; ++q) x2[((q * 4 + (c4 & 3)) * PITCH + (t >> 3) + 32 * i) * 2 + (c4 >> 2)] = s[q];
        } else if (i % 2) {
            const tdc_op3 o = tdc_split_op(x[i - 1], x[i]);
#pragma unroll
            for (int q = 0; q < 3; ++q) xb[(q * 4 + nq * (NX / 2) + i / 2) * PITCH + t % TP] = __builtin_bit_cast(tdc_u4, o.p[q]);
        }
    };

    unsigned wlane[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) wlane[mb] = mb0 + mb < a.NBm ? (unsigned)((mb0 + mb) * a.S) * 3072u + lane * 16u : TDC_OOB;
    const auto fetch_w = [&](int step_, tdc_bf8(&w)[MB][3]) {
        const int step = min(step_, a.S - 1);      // past the end: never multiplied, or (second group, odd S) with zero activations
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                w[mb][q] = __builtin_bit_cast(tdc_bf8, (tdc_u4)__builtin_amdgcn_raw_buffer_load_b128(wrs, (int)(wlane[mb] + q * 1024u), step * 3072, 0));
    };

    // NCHW y: operands swapped, so that a lane ends up with four consecutive pixels of one channel
    constexpr bool SWAP = ACT == TDC_ACT_NCHW;     // an NCHW activation means an NCHW y
    tdc_f4 acc[MB][PB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc[mb][pb] = tdc_f4_zero();
    const auto read_b = [&](const tdc_u4 *__restrict__ xb, int pb) {
        tdc_op3 b;
#pragma unroll
        for (int q = 0; q < 3; ++q) b.p[q] = __builtin_bit_cast(tdc_bf8, xb[(q * 4 + g) * PITCH + 16 * (wp * PB + pb) + l16]);
        return b;
    };
    const auto multiply = [&](int pb, const tdc_op3 &b, const tdc_bf8(&w)[MB][3]) {
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                acc[mb][pb] = SWAP ? tdc_mfma_bf(b.p[TDC_BF3_B[i]], w[mb][TDC_BF3_A[i]], acc[mb][pb])
                                   : tdc_mfma_bf(w[mb][TDC_BF3_A[i]], b.p[TDC_BF3_B[i]], acc[mb][pb]);
    };
    {
        tdc_f4 x[2][NX];
        tdc_bf8 w[2][MB][3];
        fetch_w(ks, w[0]);
        fetch_x(ks, x[0]);
        fetch_x(ks + KS, x[1]);
#pragma unroll
        for (int n = 0; n < NX; ++n) to_lds(x[0], xs[0], n);
        fetch_x(ks + 2 * KS, x[0]);
        const int steps = (a.S + KS - 1) / KS;
        for (int i = 0;; i += 2) {
            bool more = true;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (!more) break;
                __syncthreads();
                fetch_w((i + u + 1) * KS + ks, w[1 - u]);
                tdc_op3 b[2];
                b[0] = read_b(xs[u], 0);
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    if (pb + 1 < PB) b[(pb + 1) & 1] = read_b(xs[u], pb + 1);
                    multiply(pb, b[pb & 1], w[u]);
                }
#pragma unroll
                for (int n = 0; n < NX; ++n) to_lds(x[1 - u], xs[1 - u], n);
                fetch_x((i + u + 3) * KS + ks, x[1 - u]);
                // an MFMA takes 16 cycles and leaves room for two other vector instructions: the conversions of the next
                // step's activations go in between
                __builtin_amdgcn_sched_group_barrier(0x020, 3 * MB, 0);          // weights
                __builtin_amdgcn_sched_group_barrier(0x100, PB > 1 ? 6 : 3, 0);
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
#pragma unroll
                    for (int m = 0; m < 6 * MB; ++m) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
                        if (m % 4 == 3) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                        if (m == 3 * MB && pb + 2 < PB) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
                    }
                }
                more = i + u + 1 < steps;
            }
            if (!more) break;
        }
    }
    if constexpr (KS == 2) {   // the second group's sums join the first's, always in this order
        __syncthreads();
        tdc_f4 *__restrict__ red = reinterpret_cast<tdc_f4 *>(xs_all);
        static_assert(sizeof(xs_all) >= 4 * MB * PB * 64 * 16, "the partial sums fit where the activations were");
        if (ks == 1) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) red[((wave * MB + mb) * PB + pb) * 64 + lane] = acc[mb][pb];
        }
        __syncthreads();
        if (ks == 1) return;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) acc[mb][pb] += red[((wave * MB + mb) * PB + pb) * 64 + lane];
    }

    // the lane number once more: the one above need not be kept through the loop for this
    const int out_lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), og = out_lane >> 4, ol = out_lane & 15;
    // Factors without three parts, a sum that overflows on the way, or a pixel all of whose sums here are small: channels with
    // tiny weights beside others (a filter that decayed) do not make it one.
    float largest = 0.f;
    unsigned smallest = ~0u;
    const auto each_pixel = [&](auto f) {           // f(largest magnitude of this lane's channels of a pixel)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
            for (int i = 0; i < (SWAP ? 4 : 1); ++i) {
                float m = 0.f;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) m = SWAP ? __builtin_elementwise_maximum(m, fabsf(acc[mb][pb][i])) : tdc_largest(m, acc[mb][pb]);
                f(m);
            }
    };
    each_pixel([&](float m) {
        largest = __builtin_elementwise_maximum(largest, m);
        smallest = tdc_smallest(smallest, m);
    });
    bool small = false;
    if (__builtin_expect(tdc_any_lane(tdc_is_small(smallest)), 0)) {
        each_pixel([&](float m) {                   // the pixel's lanes: l16, or one lane group
            unsigned long long ok = __builtin_amdgcn_ballot_w64(!(m < TDC_SMALL));
            if (SWAP) {
                const unsigned long long low15 = 0x7fff7fff7fff7fffull;
                ok = ((((ok & low15) + low15) | ok) & ~low15) >> 15;        // bit 0 of a group: any of its lanes
                ok *= 0xffffu;
            } else {
                ok |= ok >> 32 | ok << 32;
                ok |= ok >> 16 | ok << 48;
            }
            small |= (__builtin_amdgcn_ballot_w64(m > 0.f) & ~ok) != 0;
        });
    }
    unsigned nans = 0;
    if (__builtin_expect(small || tdc_any_lane(!(largest < INFINITY)), 0))
        nans = tile_redo<ACT, CONV, MB, PB>(tdc_args_again<TileArgs>(), small, out_lane, p_base, mb0, acc);

    const auto emit = [&](int mb, int pb, tdc_f4 v) {
        if (ACT == TDC_ACT_NHWC) {
            const int p = p_base + 16 * pb + ol, m = 16 * (mb0 + mb) + 4 * og;
            if (p < a.Ptot && m < a.M) tdc_store_nhwc(a.out, a.epi, v, m, (size_t)p * a.M + m);
            return;
        }
        // four consecutive pixels of channel m
        const int p = p_base + 16 * pb + 4 * og, m = 16 * (mb0 + mb) + ol;
        if (p >= a.Ptot || m >= a.M) return;
        const int b = tdc_div(p, a.div_P), pix = p - b * a.P;
        const float bias = a.epi.bias ? a.epi.bias[m] : 0.f;
        if (a.vec) {
            const size_t idx = ((size_t)b * a.M + m) * a.P + pix;
            v += (tdc_f4){bias, bias, bias, bias};
            if (a.epi.residual) v += *reinterpret_cast<const tdc_f4 *>(a.epi.residual + idx);
            if (a.epi.relu) v = (tdc_f4){fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)};
            *reinterpret_cast<tdc_f4 *>(a.out + idx) = v;
            return;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (p + i >= a.Ptot) break;
            int bi = b, pi = pix + i;
            while (pi >= a.P) {
                pi -= a.P;
                ++bi;
            }
            const size_t idx = ((size_t)bi * a.M + m) * a.P + pi;
            float u = v[i] + bias;
            if (a.epi.residual) u += a.epi.residual[idx];
            a.out[idx] = a.epi.relu ? fmaxf(u, 0.f) : u;
        }
    };
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) emit(mb, pb, acc[mb][pb]);
    if (CONV && __builtin_expect(tdc_any_lane(nans != 0), 0)) {
        __threadfence();           // behind the stores above
        const TileArgs &args = tdc_args_again<TileArgs>();
#pragma unroll 1
        for (int e = 0; e < MB * PB * 4; ++e) {
            const int i = e & 3, pb = (e >> 2) % PB, mb = (e >> 2) / PB;
            const int p = p_base + 16 * pb + (SWAP ? 4 * og + i : ol), m = 16 * (mb0 + mb) + (SWAP ? ol : 4 * og + i);
            if ((nans >> e & 1u) && p < args.Ptot && m < args.M) tile_plain_output<ACT>(args, m, p);
        }
    }
}

template <int ACT, bool CONV>
hipError_t launch_act(const TileArgs &a, int tm, int tp, int ks, hipStream_t s)
{
    const dim3 grid((unsigned)(a.n_mt * a.n_pt));
#define TDC_CASE(M_, P_, WM_, KS_)                                                                                  \
    if (tm == M_ && tp == P_ && ks == KS_) {                                                                        \
        hipLaunchKernelGGL((tdc_tile_bf3_kernel<ACT, CONV, WM_, M_ / 16 / WM_, P_ / 16 / (4 / WM_), KS_>), grid, dim3(256 * KS_), 0, s, a); \
        return hipGetLastError();                                                                                   \
    }
    TDC_CASE(128, 64, 4, 1) TDC_CASE(64, 64, 2, 1) TDC_CASE(64, 64, 2, 2) TDC_CASE(128, 64, 4, 2)
#undef TDC_CASE
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t tdc_launch_tile_bf3(const TdcDims &d, int tm, int tp, int ks, hipStream_t s, const float *x, const void *w3, float *y, const TdcEpi &epi)
{
    TileArgs a;
    a.act = x; a.w3 = w3; a.out = y; a.epi = epi;
    a.C = d.C; a.HW = d.H * d.W; a.M = d.N; a.P = d.Ho * d.Wo; a.Ptot = d.B * a.P;
    a.NBm = d.NB2; a.NBk = d.NB1; a.KG = d.K * d.K * d.NB1; a.S = (a.KG + 1) / 2;
    a.H = d.H; a.W = d.W; a.Wo = d.Wo; a.K = d.K; a.stride = d.stride; a.pad = d.pad;
    a.n_mt = (d.N + tm - 1) / tm; a.n_pt = (a.Ptot + tp - 1) / tp;
    const size_t w_bytes = tdc_packed3_bytes(a.NBm, a.KG);
    a.w_bytes = (unsigned)w_bytes;
    a.pt_major = w_bytes < (size_t)d.B * a.C * a.HW * 4;
    a.vec = !d.nhwc && a.P % 4 == 0 && (((uintptr_t)y | (uintptr_t)epi.residual) & 15u) == 0;
    a.div_P = tdc_make_div((unsigned)a.P); a.div_Wo = tdc_make_div((unsigned)a.Wo);
    a.div_NBk = tdc_make_div((unsigned)a.NBk); a.div_K = tdc_make_div((unsigned)a.K);
    a.div_inner = tdc_make_div((unsigned)(a.pt_major ? a.n_mt : a.n_pt));
    const bool conv = d.K > 1 || d.stride > 1 || d.pad > 0;
    if (d.nhwc) return conv ? launch_act<TDC_ACT_NHWC, true>(a, tm, tp, ks, s) : launch_act<TDC_ACT_NHWC, false>(a, tm, tp, ks, s);
    return conv ? launch_act<TDC_ACT_NCHW, true>(a, tm, tp, ks, s) : launch_act<TDC_ACT_NCHW, false>(a, tm, tp, ks, s);
}
