// The dense layer for launches that are bound by matrix arithmetic or by memory bandwidth, not by latency: an implicit GEMM
//   D[m][p] = sum_k Wt[k][m] * Act[k][p]
// in TM x 64 tiles (output channels x pixels), fp32 in and out, products in two scaled fp16
// parts (tdc_split.h), three in some 1x1 layers; contractions of at most 72 terms else in three bf16 ones (tdc_tile_bf3.hip).
//
// Pixels are numbered through the whole batch, p = b*P + (pixel of image b), so small images leave no part-empty tiles.
// A workgroup is KS groups of four wavefronts; the contraction goes in steps of two 16-wide k-groups (tap, channel block),
// dealt to the groups in turn.  The activations of a step are brought in by all threads of a group, fp32 from memory (two
// steps ahead, in registers), split into their parts once and handed to the group's wavefronts through LDS, double-buffered:
// one barrier per step.  The weights were split when they were re-laid out; a wavefront loads its own fragments straight
// into registers, one step ahead.
//
// What bounds it, and why this form.  Two parts cost three products per fp32 product, 384 cycles of the matrix cores for a
// 128 x 64 step; the L1 path (24 KB a step), LDS (40 KB and its conflicts) and instruction issue (an MFMA leaves room for
// two other vector instructions: the conversions are placed between them) are then about as busy: 3x3, 128 -> 128 at 28x28,
// batch 8: 19.8 us with three bf16 parts, six products, 17.7 with two fp16 ones.  Variants of the loop as measured with the
// three bf16 parts, 128 x 64, on
// 1024 -> 512 at 14x14, batch 32 (6.6 GFLOP): both operands through LDS, two barriers a step 53 us; no LDS, every wavefront
// loading and splitting its own pixels 64 us (NHWC loads of 16 pixels x 64 bytes run at 18 bytes a cycle, a third of
// contiguous ones); this one without the interleaving 42.8 us, with it 39.8 us (fp32 MFMA kernel: 90.5 us).
#include <algorithm>
#include <cmath>

#include "tdc_split.h"
#include "tdc_internal.h"

namespace {

struct TileArgs {
    const float *act;
    const void *w;          // weights in NP parts, [NBm][S][NP][64 lanes][8 fp16] (S steps), then their exponents
    float *out;
    TdcEpi epi;             // applied where out is the layer's y
    int C;                  // channels of act
    int HW;                 // pixels per image of act
    int M;                  // output channels that exist
    int P, Ptot;            // output pixels per image, in all
    int NBm, NBk, KG, S;    // 16-blocks of M; k-groups per tap; k-groups in all; steps
    int H, W, Wo, K, stride, pad;
    int n_mt, n_pt, pt_major;
    int per, n_mg;          // 1x1: channel tiles of a workgroup, workgroups that share a pixel tile
    int half_log_terms;     // half the logarithm (2) of a sum's terms
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
    const float *w = reinterpret_cast<const float *>(tdc_raw_base(a.w, a.w_bytes, a.NBm)) + (size_t)(m >> 4) * a.KG * 256;
    float sum = 0.f;
#pragma unroll 1
    for (int kg = 0; kg < a.KG && sum == sum; ++kg) {
        const int tap = tdc_div(kg, a.div_NBk), c0 = 16 * (kg - tap * a.NBk);
        const int r = tdc_div(tap, a.div_K), h = h0 + r, wx = w0 + tap - r * a.K;
        if (h < 0 || h >= a.H || wx < 0 || wx >= a.W) continue;
        const int q = h * a.W + wx;
#pragma unroll 1
        for (int k = 0; k < 16 && c0 + k < a.C; ++k) {
            sum = fmaf(w[(size_t)kg * 256 + ((m & 15) + 16 * (k >> 2)) * 4 + (k & 3)], ACT == TDC_ACT_NHWC ? x[(size_t)q * a.C + c0 + k] : x[(size_t)(c0 + k) * a.HW + q], sum);
        }
    }
    const size_t idx = ACT == TDC_ACT_NHWC ? (size_t)p * a.M + m : ((size_t)b * a.M + m) * a.P + pix;
    a.out[idx] = tdc_apply_epilogue(a.epi, sum, m, idx);
}

// A wavefront's sums once more on the fp32 matrix cores, one load at a time (see tdc_split.h), unless their NaNs are x's or the
// weights': there is a NaN, no infinity, and everything else fits in fp16 at the scales taken.  Returns a bit per sum of this lane for those that an infinite weight at a tap outside the image made NaN (it is 0
// times the weight here, and no part of the sum).  3x3, 128 -> 128 at 28x28,
// batch 8, every value NaN: 70 us, 26 with numbers (one output after the other: 5350).
template <int ACT, bool CONV, int MB, int PB>
__device__ __forceinline__ unsigned tile_redo(const TileArgs &a, bool small, int x_exp, int lane, int p_base, int mb0, tdc_f4 (&acc)[MB][PB], bool &done)
{
    constexpr bool SWAP = ACT == TDC_ACT_NCHW;
    const int g = lane >> 4, l16 = lane & 15;
    const int b0 = tdc_div(p_base, a.div_P), n_img = min((16 * PB - 1) / a.P + 2, tdc_div(a.Ptot - 1, a.div_P) + 1 - b0);
    const size_t img_elems = (size_t)a.C * a.HW;
    const tdc_rsrc ars = tdc_make_rsrc(a.act + (size_t)b0 * img_elems, (unsigned)(n_img * img_elems * 4));
    const tdc_rsrc wrs = tdc_make_rsrc(tdc_raw_base(a.w, a.w_bytes, a.NBm), 1024u * a.NBm * a.KG);
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
    const auto load_w = [&](int kg, int mb) { return mb0 + mb < a.NBm ? tdc_raw_weights(wrs, mb0 + mb, a.KG, kg, lane) : tdc_f4_zero(); };

    TdcFactors xs, ws;
#pragma unroll 2
    for (int kg = 0; kg < a.KG; ++kg) {
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) xs.see(load_x(kg, pb));
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            ws.see(load_w(kg, mb));
    }
    const bool odd_weights = tdc_any_lane(ws.nan || ws.largest == INFINITY);
    bool in_parts = true;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) in_parts &= !tdc_any_lane(mb0 + mb < a.NBm && reinterpret_cast<const int *>(static_cast<const char *>(a.w) + a.w_bytes)[16 * min(mb0 + mb, a.NBm - 1) + l16] == TDC_WIDE);
    const bool explained = in_parts && tdc_any_lane(xs.nan | ws.nan) && !tdc_any_lane(ldexpf(xs.largest, x_exp) > TDC_FP16_MAX || ws.largest == INFINITY);
    done = !(explained && !small && !(CONV && odd_weights));
    if (!done) return 0u;

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

// The largest magnitude of each of a tile's 64 pixels, from the threads that brought it: in NHWC eight lanes share a pixel of every 32,
// in NCHW four wavefronts share all.  ROWS: what is kept apart until all have written.
constexpr int tile_top_rows(int act, int ks) { return act == TDC_ACT_NHWC ? ks : 4 * ks; }
template <bool NHWC, int NPIX>
__device__ __forceinline__ void tile_put_tops(const float (&x_top)[NPIX], float (*__restrict__ tops)[64], int ks, int t)
{
    if (!NHWC) {
        tops[4 * ks + (t >> 6)][t & 63] = x_top[0];
        return;
    }
#pragma unroll
    for (int i = 0; i < NPIX; ++i) {
        unsigned u = __builtin_bit_cast(unsigned, x_top[i]);
        u = max(u, (unsigned)__builtin_amdgcn_mov_dpp((int)u, 0xb1, 0xf, 0xf, true));      // quad_perm 1 0 3 2
        u = max(u, (unsigned)__builtin_amdgcn_mov_dpp((int)u, 0x4e, 0xf, 0xf, true));      // quad_perm 2 3 0 1
        u = max(u, (unsigned)__builtin_amdgcn_mov_dpp((int)u, 0x141, 0xf, 0xf, true));     // the other half of eight
        if ((t & 7) == 0) tops[ks][(t >> 3) + 32 * i] = __builtin_bit_cast(float, u);
    }
}
// a wavefront's, a pixel to a lane
template <int ROWS>
__device__ __forceinline__ unsigned tile_top(const float (*__restrict__ tops)[64], int lane)
{
    unsigned u = 0;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) u = max(u, __builtin_bit_cast(unsigned, tops[i][lane]));
    return u;
}
// whether there is a pixel of nothing but values too small for all their bits
__device__ __forceinline__ bool tile_too_small(unsigned top, int x_exp)
{
    return tdc_any_lane(tdc_is_small(tdc_smallest(~0u, __builtin_bit_cast(float, top)), tdc_exp2i(max(TDC_LOWEST - x_exp, -126))));
}

// What a channel's largest sum among a lane's pixels must reach, as bits: 2^22 times what the parts lose.  With scaled weights of 2^12
// root mean square, x up to `top` times 2^x_exp and 2^(2 half_log_terms) terms two parts lose sqrt(terms) (2^-25 + 2^-39 x), of
// three, where the weights' are not lifted, sqrt(terms) (2^-25 + 2^-28 x).  Normal values give 2^18 (2^15) times more.
template <int NP>
__device__ __forceinline__ int tile_lost(int half_log_terms, unsigned top, int x_exp)
{
    const int e = min((int)(top >> 23) - 126 + x_exp, 16);
    return (127 + half_log_terms + max(-2, e - (NP == 2 ? 17 : 6))) << 23;
}
// The magnitudes of a wavefront's sums: of all the largest, NaN if there is one, and of the channels' largest the least, as bits.
template <bool SWAP, int MB, int PB>
__device__ __forceinline__ void tile_magnitudes(const tdc_f4 (&acc)[MB][PB], float &largest, int &least)
{
    largest = 0.f;
    least = 0x7f800000;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int c = 0; c < (SWAP ? 1 : 4); ++c) {
            float m = 0.f;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int i = SWAP ? 0 : c; i < (SWAP ? 4 : c + 1); ++i) m = __builtin_elementwise_maximum(m, fabsf(acc[mb][pb][i]));
            largest = __builtin_elementwise_maximum(largest, m);
            least = min(least, __builtin_bit_cast(int, m));
        }
}
// Whether a wavefront lost a channel: the least once more, of `blocks` channel blocks and of sums that are no NaN, over the pixels of
// lanes that are put together until some have four at which x is not all zero: fewer sums may be small by chance.  top: tile_top;
// first: the wavefront's first pixel.
template <bool SWAP, int MB, int PB>
__device__ __forceinline__ bool tile_lost_any(const tdc_f4 (&acc)[MB][PB], int blocks, unsigned top, int first, int lane, int lost)
{
    constexpr int NEXT = SWAP ? 16 : 8, END = SWAP ? 64 : 0;       // a lane holds four pixels of each block, or one
    const auto further = [](int step) { return SWAP ? 2 * step : step / 2; };
    const unsigned long long px = __builtin_amdgcn_ballot_w64(top != 0) >> first;
    int lit = 0;
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) lit += SWAP ? __builtin_popcount((unsigned)(px >> 16 * pb) >> 4 * (lane >> 4) & 15u) : (int)(px >> (16 * pb + (lane & 15)) & 1u);
    int end = NEXT;                                                 // all steps in front of it are taken
    do {
        lit += __shfl_xor(lit, end);
        end = further(end);
    } while (end != END && !tdc_any_lane(lit > 3));
    int least = 0x7f800000;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int c = 0; c < (SWAP ? 1 : 4); ++c) {
            float m = -1.f;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int i = SWAP ? 0 : c; i < (SWAP ? 4 : c + 1); ++i) m = fmaxf(m, fabsf(acc[mb][pb][i]));
#pragma unroll 1
            for (int step = NEXT; step != end; step = further(step)) m = fmaxf(m, __shfl_xor(m, step));
            if (m >= 0.f && mb < blocks) least = min(least, __builtin_bit_cast(int, m));
        }
    return tdc_any_lane(lit > (tdc_any_lane(lit > 3) ? 3 : 0) && least < lost);
}

// Four pixels of NCHW channel m, from pixel p on, that cannot be stored at once: sums and bias in v, shortcut and ReLU here.
__device__ __forceinline__ void tile_store_4(const TileArgs &a, tdc_f4 v, int p, int m)
{
    if (p >= a.Ptot) return;
    int b = tdc_div(p, a.div_P), pix = p - b * a.P;
#pragma unroll
    for (int i = 0; i < 4; ++i, ++pix) {
        if (p + i >= a.Ptot) break;
        while (pix >= a.P) {
            pix -= a.P;
            ++b;
        }
        const size_t idx = ((size_t)b * a.M + m) * a.P + pix;
        float u = v[i];
        if (a.epi.residual) u += a.epi.residual[idx];
        a.out[idx] = a.epi.relu ? fmaxf(u, 0.f) : u;
    }
}

// Wavefronts per SIMD an instance has registers for.
constexpr int tile_wavefronts(int mb_pb) { return mb_pb > 4 ? 2 : 3; }

template <int ACT, bool CONV, int WM, int MB, int PB, int KS>
__global__ __launch_bounds__(256 * KS, tile_wavefronts(MB * PB)) void tdc_tile_kernel(TileArgs a)
{
    constexpr int NP = 2;                          // parts
    constexpr int WP = 4 / WM, TM = 16 * MB * WM, TP = 16 * PB * WP;
    constexpr int NX = TP / 32;                    // 16-byte pieces of activations a thread brings per step
    constexpr int PITCH = TP + 4;                  // 16-byte cells
    constexpr int NM = TdcProducts<NP>::N;
    constexpr int VPM = (NX * (7 * NP + (ACT == TDC_ACT_NCHW ? 17 : 12)) + 20 + NM * MB * PB - 1) / (NM * MB * PB);   // VALU instructions per MFMA
    __shared__ tdc_u4 xs_all[KS][2][4 * NP * PITCH];   // [part][lane group][pixel]: 4 channels of each k-group of the step
    __shared__ unsigned first_all[4 * KS];             // largest magnitude among what each wavefront loads first
    constexpr int TOP_ROWS = tile_top_rows(ACT, KS);
    __shared__ float tops[TOP_ROWS][64];               // largest magnitudes of the pixels
    const int ks = KS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
    tdc_u4(&xs)[2][4 * NP * PITCH] = xs_all[ks];
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
    const tdc_rsrc wrs = tdc_make_rsrc(a.w, a.w_bytes);

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
    int x_exp = 0;                                 // x is multiplied by 2^x_exp
    float x_top[NPIX] = {};                        // largest magnitude of what this thread has brought of a pixel
    const auto to_lds = [&](const tdc_f4(&x)[NX], tdc_u4 *__restrict__ xb, int i) {
        const TdcScale scale(x_exp);
        x_top[i % NPIX] = tdc_largest(x_top[i % NPIX], x[i]);
        if (ACT == TDC_ACT_NHWC) {
            tdc_u2 *__restrict__ x2 = reinterpret_cast<tdc_u2 *>(xb);
            tdc_u2 s[NP];
            tdc_split4<NP>(x[i], scale, s);
#pragma unroll
            for (int q = 0; q < NP; ++q) x2[((q * 4 + (c4 & 3)) * PITCH + (t >> 3) + 32 * i) * 2 + (c4 >> 2)] = s[q];
        } else if (i % 2) {
            const tdc_op<NP> o = tdc_split_op<NP>(x[i - 1], x[i], scale);
#pragma unroll
            for (int q = 0; q < NP; ++q) xb[(q * 4 + nq * (NX / 2) + i / 2) * PITCH + t % TP] = __builtin_bit_cast(tdc_u4, o.p[q]);
        }
    };

    unsigned wlane[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) wlane[mb] = mb0 + mb < a.NBm ? (unsigned)((mb0 + mb) * a.S) * (1024u * NP) + lane * 16u : TDC_OOB;
    const auto fetch_w = [&](int step_, tdc_op<NP>(&w)[MB]) {
        const int step = min(step_, a.S - 1);      // past the end: never multiplied, or (second group, odd S) with zero activations
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int q = 0; q < NP; ++q)
                w[mb].p[q] = __builtin_bit_cast(tdc_h8, (tdc_u4)__builtin_amdgcn_raw_buffer_load_b128(wrs, (int)(wlane[mb] + q * 1024u), step * (1024 * NP), 0));
    };

    // NCHW y: operands swapped, so that a lane ends up with four consecutive pixels of one channel
    constexpr bool SWAP = ACT == TDC_ACT_NCHW;     // an NCHW activation means an NCHW y
    tdc_f4 lev[MB][PB][TDC_LEVELS];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
            for (int q = 0; q < TDC_LEVELS; ++q) lev[mb][pb][q] = tdc_f4_zero();
    const auto read_b = [&](const tdc_u4 *__restrict__ xb, int pb) {
        tdc_op<NP> b;
#pragma unroll
        for (int q = 0; q < NP; ++q) b.p[q] = __builtin_bit_cast(tdc_h8, xb[(q * 4 + g) * PITCH + 16 * (wp * PB + pb) + l16]);
        return b;
    };
    const auto multiply = [&](int pb, const tdc_op<NP> &b, const tdc_op<NP>(&w)[MB]) {
#pragma unroll
        for (int i = 0; i < NM; ++i)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                tdc_f4 &c = lev[mb][pb][TdcProducts<NP>::level[i]];
                c = tdc_mfma_part<NP, SWAP>(i, w[mb].p, b.p, c);
            }
    };
    // Exponents of the lane's output channels: here and not behind the loop, where nothing would hide their way (3x3, 128 -> 128 at
    // 28x28, batch 8: 17.8 -> 17.2 us; 33 drawn NCHW layers 1.2 %), but in NHWC with two groups of wavefronts, 1 % slower so.
    constexpr bool EARLY = SWAP || KS == 1;
    int w_exp[MB][SWAP ? 1 : 4];
    const auto fetch_exponents = [&](int row, int col) {
        const int *__restrict__ exponents = reinterpret_cast<const int *>(static_cast<const char *>(a.w) + a.w_bytes);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < (SWAP ? 1 : 4); ++i) w_exp[mb][i] = exponents[16 * min(mb0 + mb, a.NBm - 1) + (SWAP ? col : 4 * row + i)];
    };
    if (EARLY) fetch_exponents(g, l16);
    {
        tdc_f4 x[2][NX];
        tdc_op<NP> w[2][MB];
        fetch_w(ks, w[0]);
        fetch_x(ks, x[0]);
        fetch_x(ks + KS, x[1]);
        float m = 0.f;
#pragma unroll
        for (int n = 0; n < NX; ++n) m = tdc_largest_number(m, x[0][n]);
        first_all[4 * ks + wave] = tdc_wave_max(m);
        __syncthreads();
        unsigned first = 0;
#pragma unroll
        for (int i = 0; i < 4 * KS; ++i) first = max(first, first_all[i]);
        x_exp = tdc_scale_of((unsigned)__builtin_amdgcn_readfirstlane((int)first), TDC_X_TARGET, TDC_X_OTHER);
        if (EARLY) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < (SWAP ? 1 : 4); ++i) asm volatile("" : "+v"(w_exp[mb][i]));     // they came before x
        }
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
                tdc_op<NP> b[2];
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
                __builtin_amdgcn_sched_group_barrier(0x020, NP * MB, 0);          // weights
                __builtin_amdgcn_sched_group_barrier(0x100, PB > 1 ? 2 * NP : NP, 0);
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
#pragma unroll
                    for (int m = 0; m < NM * MB; ++m) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
                        if (m % 4 == 3) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                        if (m == NM / 2 * MB && pb + 2 < PB) __builtin_amdgcn_sched_group_barrier(0x100, NP, 0);
                    }
                }
                more = i + u + 1 < steps;
            }
            if (!more) break;
        }
    }
    tile_put_tops<ACT == TDC_ACT_NHWC, NPIX>(x_top, tops, ks, t);
    tdc_f4 acc[MB][PB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc[mb][pb] = tdc_levels(lev[mb][pb]);
    if (KS == 1) __syncthreads();
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
    // factors too small, too large or without a value
    float largest;
    int least;
    tile_magnitudes<SWAP, MB, PB>(acc, largest, least);
    const unsigned top = tile_top<TOP_ROWS>(tops, out_lane);
    const int lost = tile_lost<NP>(a.half_log_terms, tdc_wave_max(__builtin_bit_cast(float, top)), x_exp);
    bool small = tile_too_small(top, x_exp);
    if (!EARLY) fetch_exponents(og, ol);
    unsigned nans = 0;
    bool redone = false;
    if (__builtin_expect(small || tdc_any_lane(!tdc_finite(largest) || least < lost), 0)) {
        small = small || tile_lost_any<SWAP, MB, PB>(acc, a.NBm - mb0, top, 16 * PB * wp, out_lane, lost);
        if (small || tdc_any_lane(!tdc_finite(largest)))
            nans = tile_redo<ACT, CONV, MB, PB>(tdc_args_again<TileArgs>(), small, x_exp, out_lane, p_base, mb0, acc, redone);
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        if (redone || mb0 + mb >= a.NBm) break;
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[mb][pb][i] = ldexpf(acc[mb][pb][i], -x_exp - w_exp[mb][SWAP ? 0 : i]);
    }

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
        tile_store_4(a, v + (tdc_f4){bias, bias, bias, bias}, p, m);
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

// ---- 1x1 layers whose whole contraction fits in LDS
//
// A workgroup brings its 64 pixels once, all channels, split, into LDS, and then runs over `per` tiles of 64 MB output channels: no
// barrier between them, weights one step ahead across the tiles, bias and shortcut of a tile in flight under its products.
template <int ACT, int MB, int NP>
__global__ __launch_bounds__(256, MB == 2 ? 2 : 3) void tdc_tile_1x1_kernel(TileArgs a)
{
    constexpr bool NHWC = ACT == TDC_ACT_NHWC, SWAP = !NHWC;
    constexpr int PB = 4, TP = 16 * PB, PITCH = TP + 4, NX = 2, NM = TdcProducts<NP>::N, CHUNK = 4;
    constexpr int STEP = 4 * NP * PITCH;               // 16-byte cells of a step: [part][lane group][pixel]
    extern __shared__ tdc_u4 tile_1x1_lds[];
    constexpr int TOP_ROWS = tile_top_rows(ACT, 1);
    unsigned *__restrict__ first_all = reinterpret_cast<unsigned *>(tile_1x1_lds);               // four first magnitudes, then
    float(*__restrict__ tops)[64] = reinterpret_cast<float(*)[64]>(tile_1x1_lds + 1);            // largest ones of the pixels
    tdc_u4 *__restrict__ xs = tile_1x1_lds + 1 + TOP_ROWS * 16;
    const int t = threadIdx.x, lane = t & 63, g = lane >> 4, l16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int lb = tile_logical_block(blockIdx.x, gridDim.x);
    const int pt = tdc_div(lb, a.div_inner), mt0 = (lb - pt * a.n_mg) * a.per, mt1 = min(mt0 + a.per, a.n_mt);
    const int p_tile = pt * TP;
    const int b0 = tdc_div(p_tile, a.div_P);
    const size_t img_elems = (size_t)a.C * a.HW;
    const int n_img = min((TP - 1) / a.P + 2, tdc_div(a.Ptot - 1, a.div_P) + 1 - b0);
    const tdc_rsrc ars = tdc_make_rsrc(a.act + (size_t)b0 * img_elems, (unsigned)(n_img * img_elems * 4));
    const tdc_rsrc wrs = tdc_make_rsrc(a.w, a.w_bytes + 64u * a.NBm);       // with the exponents

    const auto fetch_w = [&](int mt, int step, tdc_op<NP>(&w)[MB]) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int blk = (mt * 4 + wave) * MB + mb;
            const unsigned o = blk < a.NBm && mt < mt1 ? (unsigned)(blk * a.S + step) * (1024u * NP) + lane * 16u : TDC_OOB;
#pragma unroll
            for (int q = 0; q < NP; ++q) w[mb].p[q] = __builtin_bit_cast(tdc_h8, tdc_buf_load4(wrs, o + q * 1024u));
        }
    };
    tdc_op<NP> w0[MB];
    fetch_w(mt0, 0, w0);

    // ---- the pixels: NHWC: a thread brings four channels of one pixel in 8 of each, NCHW: 4 NX channels of one pixel
    int x_exp;
    {
        constexpr int NPIX = NHWC ? NX : 1;
        const int c4 = t & 7, nq = t / TP;
        unsigned poff[NPIX];
#pragma unroll
        for (int i = 0; i < NPIX; ++i) {
            const int p = p_tile + (NHWC ? (t >> 3) + 32 * i : t % TP);
            const int b = tdc_div(p < a.Ptot ? p : p_tile, a.div_P), pix = p - b * a.P;
            poff[i] = p < a.Ptot ? (unsigned)((b - b0) * (int)img_elems + (NHWC ? pix * a.C + 4 * c4 : pix + 2 * NX * nq * a.HW)) * 4u : TDC_OOB;
        }
        const auto fetch_x = [&](int step, tdc_f4(&x)[NX]) {
            const unsigned dead = (unsigned)(a.S - 1 - step) & TDC_OOB;
            if (NHWC) {
                const unsigned bad = dead | ((unsigned)(a.C - 1 - 32 * step - 4 * c4) & TDC_OOB);
#pragma unroll
                for (int i = 0; i < NX; ++i) x[i] = tdc_buf_load4(ars, (poff[i] + 128u * step) | bad | (poff[i] & TDC_OOB));
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int c = 32 * step + 16 * h, left = a.C - 1 - c - 2 * NX * nq;   // this thread's last channel that exists
                    const unsigned o = (poff[0] + (unsigned)(c * a.HW) * 4u) | dead | (poff[0] & TDC_OOB);
#pragma unroll
                    for (int n = 0; n < NX / 2; ++n)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            x[2 * n + h][j] = tdc_buf_load(ars, (o + (unsigned)((4 * n + j) * a.HW) * 4u) | ((o | (unsigned)(left - 4 * n - j)) & TDC_OOB));
                }
            }
        };
        float x_top[NPIX] = {};
        const auto to_lds = [&](const tdc_f4(&x)[NX], const TdcScale &scale, int step) {
            if (step >= a.S) return;
            tdc_u4 *__restrict__ xb = xs + step * STEP;
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                x_top[i % NPIX] = tdc_largest(x_top[i % NPIX], x[i]);
                if (NHWC) {
                    tdc_u2 *__restrict__ x2 = reinterpret_cast<tdc_u2 *>(xb);
                    tdc_u2 s[NP];
                    tdc_split4<NP>(x[i], scale, s);
#pragma unroll
                    for (int q = 0; q < NP; ++q) x2[((q * 4 + (c4 & 3)) * PITCH + (t >> 3) + 32 * i) * 2 + (c4 >> 2)] = s[q];
                } else if (i % 2) {
                    const tdc_op<NP> o = tdc_split_op<NP>(x[i - 1], x[i], scale);
#pragma unroll
                    for (int q = 0; q < NP; ++q) xb[(q * 4 + nq * (NX / 2) + i / 2) * PITCH + t % TP] = __builtin_bit_cast(tdc_u4, o.p[q]);
                }
            }
        };
        tdc_f4 x[CHUNK][NX];
#pragma unroll
        for (int u = 0; u < CHUNK; ++u) fetch_x(u, x[u]);
        float m = 0.f;
#pragma unroll
        for (int u = 0; u < CHUNK; ++u)
#pragma unroll
            for (int n = 0; n < NX; ++n) m = tdc_largest_number(m, x[u][n]);
        first_all[wave] = tdc_wave_max(m);
        __syncthreads();
        const tdc_u4 first = tile_1x1_lds[0];
        x_exp = tdc_scale_of((unsigned)__builtin_amdgcn_readfirstlane((int)max(max(first[0], first[1]), max(first[2], first[3]))), TDC_X_TARGET, TDC_X_OTHER);
        const TdcScale scale(x_exp);
        for (int s = 0; s < a.S; s += CHUNK) {
#pragma unroll
            for (int u = 0; u < CHUNK; ++u) {
                to_lds(x[u], scale, s + u);
                if (s + CHUNK < a.S) fetch_x(s + CHUNK + u, x[u]);
            }
        }
        tile_put_tops<NHWC, NPIX>(x_top, tops, 0, t);
    }
    __syncthreads();
    const unsigned top = tile_top<TOP_ROWS>(tops, lane);
    const bool small = tile_too_small(top, x_exp);
    const int lost = tile_lost<NP>(a.half_log_terms, tdc_wave_max(__builtin_bit_cast(float, top)), x_exp);

    // ---- where this lane's outputs are: NHWC: channels 4g.. of pixel l16 of block pb, NCHW: pixels 4g.. of channel l16
    // (bytes from the tile's first pixel or image on; two images, or what a tile spans of smaller ones, are below 4 GiB)
    constexpr unsigned NOWHERE = ~0u;
    const size_t base = NHWC ? (size_t)p_tile * a.M : (size_t)b0 * a.M * a.P;
    char *__restrict__ out = reinterpret_cast<char *>(a.out + base);
    const char *__restrict__ shortcut = reinterpret_cast<const char *>(a.epi.residual + base);
    unsigned out_at[PB];
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        const int p = p_tile + 16 * pb + (NHWC ? l16 : 4 * g);
        const int b = tdc_div(p, a.div_P);
        out_at[pb] = p >= a.Ptot ? NOWHERE : 4u * (NHWC ? (unsigned)((p - p_tile) * a.M) : (unsigned)(b - b0) * (unsigned)(a.M * a.P) + (unsigned)(p - b * a.P));
    }
    const bool quads = NHWC || a.vec;                  // outputs go out, and shortcuts come in, 16 bytes at a time
    for (int mt = mt0; mt < mt1; ++mt) {
        const int blk0 = (mt * 4 + wave) * MB;
        // exponents, bias and shortcut of this tile, under its products
        int e[MB][NHWC ? 4 : 1];
        tdc_f4 bias[MB], res[MB][PB];
        const bool with_res = quads && a.epi.residual;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = 16 * (blk0 + mb) + (NHWC ? 4 * g : l16);
            const bool live = m < a.M;
            if (NHWC) {
                const tdc_u4 u = __builtin_bit_cast(tdc_u4, tdc_buf_load4(wrs, a.w_bytes + 4u * m));
#pragma unroll
                for (int i = 0; i < 4; ++i) e[mb][i % (NHWC ? 4 : 1)] = (int)u[i];
                bias[mb] = a.epi.bias && live ? (tdc_f4){a.epi.bias[m], a.epi.bias[m + 1], a.epi.bias[m + 2], a.epi.bias[m + 3]} : tdc_f4_zero();
            } else {
                e[mb][0] = __builtin_amdgcn_raw_buffer_load_b32(wrs, (int)(a.w_bytes + 4u * m), 0, 0);
                bias[mb][0] = a.epi.bias && live ? a.epi.bias[m] : 0.f;
            }
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
                res[mb][pb] = with_res && live && out_at[pb] != NOWHERE ? *reinterpret_cast<const tdc_f4 *>(shortcut + (out_at[pb] + 4u * (NHWC ? m : m * a.P))) : tdc_f4_zero();
        }
        tdc_f4 lev[MB][PB][TDC_LEVELS];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int q = 0; q < TDC_LEVELS; ++q) lev[mb][pb][q] = tdc_f4_zero();
        for (int s = 0; s < a.S; ++s) {
            tdc_op<NP> w1[MB];
            const bool turn = s + 1 == a.S;
            fetch_w(turn ? mt + 1 : mt, turn ? 0 : s + 1, w1);
            const tdc_u4 *__restrict__ xb = xs + s * STEP;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                tdc_op<NP> b;
#pragma unroll
                for (int q = 0; q < NP; ++q) b.p[q] = __builtin_bit_cast(tdc_h8, xb[(q * 4 + g) * PITCH + 16 * pb + l16]);
#pragma unroll
                for (int i = 0; i < NM; ++i)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) {
                        tdc_f4 &c = lev[mb][pb][TdcProducts<NP>::level[i]];
                        c = tdc_mfma_part<NP, SWAP>(i, w0[mb].p, b.p, c);
                    }
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) w0[mb] = w1[mb];
        }
        float largest;
        int least;
        tdc_f4 acc[MB][PB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) acc[mb][pb] = tdc_levels(lev[mb][pb]);
        tile_magnitudes<SWAP, MB, PB>(acc, largest, least);
        bool redone = false;
        if (__builtin_expect(small || tdc_any_lane(!tdc_finite(largest) || least < lost), 0)) {
            const bool too_small = small || tile_lost_any<SWAP, MB, PB>(acc, a.NBm - blk0, tile_top<TOP_ROWS>(tops, lane), 0, lane, lost);
            if (too_small || tdc_any_lane(!tdc_finite(largest)))
                tile_redo<ACT, false, MB, PB>(tdc_args_again<TileArgs>(), too_small, x_exp, lane, p_tile, blk0, acc, redone);
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = 16 * (blk0 + mb) + (NHWC ? 4 * g : l16);
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                tdc_f4 v = acc[mb][pb];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = redone ? v[i] : ldexpf(v[i], -x_exp - e[mb][NHWC ? i : 0]);
                    v[i] += bias[mb][NHWC ? i : 0];
                    v[i] += res[mb][pb][i];
                }
                if (quads) {
                    if (a.epi.relu) v = (tdc_f4){fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)};
                    if (m < a.M && out_at[pb] != NOWHERE) *reinterpret_cast<tdc_f4 *>(out + (out_at[pb] + 4u * (NHWC ? m : m * a.P))) = v;
                } else if (m < a.M) {
                    tile_store_4(a, v, p_tile + 16 * pb + 4 * g, m);
                }
            }
        }
    }
}

template <int ACT, bool CONV>
hipError_t launch_act(const TileArgs &a, int tm, int tp, int ks, hipStream_t s)
{
    const dim3 grid((unsigned)(a.n_mt * a.n_pt));
#define TDC_CASE(M_, P_, WM_, KS_)                                                                                   \
    if (tm == M_ && tp == P_ && ks == KS_) {                                                                        \
        hipLaunchKernelGGL((tdc_tile_kernel<ACT, CONV, WM_, M_ / 16 / WM_, P_ / 16 / (4 / WM_), KS_>), grid, dim3(256 * KS_), 0, s, a); \
        return hipGetLastError();                                                                                   \
    }
    TDC_CASE(128, 64, 4, 1) TDC_CASE(64, 64, 2, 1) TDC_CASE(64, 64, 2, 2) TDC_CASE(128, 64, 4, 2)
#undef TDC_CASE
    return hipErrorInvalidValue;
}

// LDS of the 1x1 kernel, and the most that still leaves two workgroups on a compute unit.
size_t tile_1x1_lds_bytes(int steps, int parts, bool nhwc) { return 16 + 256 * (size_t)(nhwc ? 1 : 4) + (size_t)steps * parts * 4 * 68 * 16; }
constexpr size_t TILE_1X1_LDS = 80 * 1024;

// Channel tiles a workgroup takes: the share with the shortest schedule, in channel tiles of one workgroup.  Bringing the pixels
// costs 0.3 of one; a compute unit works on `slots` workgroups at a time (registers, LDS); fewer than that at the end leave it
// partly idle, a lone one for 1.6 times its work.  us for shares of 1 / 2 / 4 / 8: 128 -> 512 at 28x28, batch 32: 38.3 / 37.4 /
// 42.0 / 37.3; 256 -> 1024 at 14x14: 25.0 / 21.5 / 28.2 / 48.4; 64 -> 256 at 56x56: 67.3 / 62.7 / 63.2 (four are all).
int tile_1x1_share(int n_pt, int n_mt, int mb, size_t lds)
{
    constexpr int cus = 256;
    const int slots = std::min(mb == 2 ? 2 : 3, (int)(160 * 1024 / lds));
    int best = 1;
    double best_time = 1e300;
    for (int per = 1; per <= n_mt; ++per) {
        const long wgs = (long)n_pt * ((n_mt + per - 1) / per), rounds = wgs / (cus * slots), rest = (wgs - rounds * cus * slots + cus - 1) / cus;
        const double time = (per + 0.3) * (rounds * slots + (rest ? std::max(1.6, (double)rest) : 0.0));
        if (time < best_time) {
            best = per;
            best_time = time;
        }
    }
    return best;
}

template <int ACT>
hipError_t launch_1x1(const TileArgs &a, int mb, int parts, hipStream_t s, bool prepare_only)
{
    const dim3 grid((unsigned)(a.n_pt * a.n_mg));
    const size_t lds = tile_1x1_lds_bytes(a.S, parts, ACT == TDC_ACT_NHWC);
    const auto kernel = parts == 3 ? tdc_tile_1x1_kernel<ACT, 1, 3> : mb == 1 ? tdc_tile_1x1_kernel<ACT, 1, 2> : tdc_tile_1x1_kernel<ACT, 2, 2>;
    const hipError_t e = tdc_allow_lds((const void *)kernel, lds);
    if (e != hipSuccess || prepare_only) return e;
    hipLaunchKernelGGL(kernel, grid, dim3(256), lds, s, a);
    return hipGetLastError();
}

}  // namespace

bool tdc_tile_supported(int tm, int tp, int ks) { return tp == 64 && (tm == 64 || tm == 128) && (ks == 1 || ks == 2); }

// Everything the kernel addresses relative to one descriptor must lie within 2 GiB of its base.
bool tdc_tile_applies(const TdcDims &d)
{
    constexpr int tp = 64;
    const size_t img = (size_t)d.C * d.H * d.W * 4, P = (size_t)d.Ho * d.Wo;
    const size_t w = tdc_packed3_bytes(d.NB2, d.K * d.K * d.NB1);      // the largest of the forms, and than what lies behind any parts
    return ((tp - 1) / P + 2) * img < (1ull << 31) && w < (1ull << 31) && (size_t)d.B * P < (1ull << 31) - 1024;
}

bool tdc_tile_1x1_applies(const TdcDims &d)
{
    const int parts = tdc_tile_parts(d);
    if (tdc_split_bytes(parts, d.NB2, d.NB1) + (size_t)64 * d.NB2 >= 1ull << 31) return false;      // with the exponents
    if (d.K != 1 || d.stride != 1 || d.pad != 0 || !tdc_tile_applies(d) || tile_1x1_lds_bytes((d.NB1 + 1) / 2, parts, d.nhwc) > TILE_1X1_LDS) return false;
    // Timed against the tile kernels on 121 drawn layers.  NCHW pixels that allow no 16-byte stores were slower in all of 40 (64 -> 368, 80
    // against 110 us).  Three parts pay from 128 output channels and 3.3 tiles per compute unit on (56 -> 64, batch-bound: 14.5 against
    // 16.1; 56 -> 140 with 3 tiles: 7.6 against 9.2; 70 -> 192 with 15: 39.6 against 33.0).  The pixels come in before the first product: with
    // many channels that has to pay for several channel tiles (256 -> 56: 12.5 against 16.1; 260 -> 164: 30.2 against 35.9;
    // NCHW 243 -> 44: 29.2 against 33.5; 228 -> 96: 26.8 against 22.9; 288 -> 384: 35.4 against 31.9).
    if (!d.nhwc && (d.Ho * d.Wo) % 4) return false;
    if (parts == 3) return d.N >= 128 && (double)((d.B * d.Ho * d.Wo + 63) / 64) * ((d.N + 63) / 64) >= 3.3 * 256;
    return d.R1 <= (d.nhwc ? 200 : 144) || (d.N > 64 && d.R1 <= 256) || d.N > 256;
}

hipError_t tdc_launch_tile_dense(const TdcDims &d, int tm, int tp, int ks, hipStream_t s, const float *x, const void *w, float *y, const TdcEpi &epi, bool prepare_only)
{
    if (prepare_only && !(ks == 1 && tdc_tile_1x1_applies(d))) return hipSuccess;      // nothing to set up
    TileArgs a;
    a.act = x; a.w = w; a.out = y; a.epi = epi;
    a.C = d.C; a.HW = d.H * d.W; a.M = d.N; a.P = d.Ho * d.Wo; a.Ptot = d.B * a.P;
    a.NBm = d.NB2; a.NBk = d.NB1; a.KG = d.K * d.K * d.NB1; a.S = (a.KG + 1) / 2;
    a.H = d.H; a.W = d.W; a.Wo = d.Wo; a.K = d.K; a.stride = d.stride; a.pad = d.pad;
    a.n_mt = (d.N + tm - 1) / tm; a.n_pt = (a.Ptot + tp - 1) / tp;
    const int parts = tdc_tile_parts(d);
    if (tdc_tile_bf3(d, ks)) return tdc_launch_tile_bf3(d, tm, tp, ks, s, x, w, y, epi);
    const size_t w_bytes = tdc_split_bytes(parts, a.NBm, a.KG);
    a.w_bytes = (unsigned)w_bytes;
    a.pt_major = w_bytes < (size_t)d.B * a.C * a.HW * 4;
    a.half_log_terms = (int)std::lround(0.5 * std::log2((double)d.K * d.K * d.C));
    a.vec = !d.nhwc && a.P % 4 == 0 && (((uintptr_t)y | (uintptr_t)epi.residual) & 15u) == 0;
    a.div_P = tdc_make_div((unsigned)a.P); a.div_Wo = tdc_make_div((unsigned)a.Wo);
    a.div_NBk = tdc_make_div((unsigned)a.NBk); a.div_K = tdc_make_div((unsigned)a.K);
    a.div_inner = tdc_make_div((unsigned)(a.pt_major ? a.n_mt : a.n_pt));
    const bool conv = d.K > 1 || d.stride > 1 || d.pad > 0;
    if (ks == 1 && tdc_tile_1x1_applies(d)) {
        const int mb = parts == 3 ? 1 : tm / 64;
        a.n_mt = (d.N + 64 * mb - 1) / (64 * mb);
        a.per = tile_1x1_share(a.n_pt, a.n_mt, mb, tile_1x1_lds_bytes(a.S, parts, d.nhwc));
        a.n_mg = (a.n_mt + a.per - 1) / a.per;
        a.div_inner = tdc_make_div((unsigned)a.n_mg);
        return d.nhwc ? launch_1x1<TDC_ACT_NHWC>(a, mb, parts, s, prepare_only) : launch_1x1<TDC_ACT_NCHW>(a, mb, parts, s, prepare_only);
    }
    if (d.nhwc) return conv ? launch_act<TDC_ACT_NHWC, true>(a, tm, tp, ks, s) : launch_act<TDC_ACT_NHWC, false>(a, tm, tp, ks, s);
    return conv ? launch_act<TDC_ACT_NCHW, true>(a, tm, tp, ks, s) : launch_act<TDC_ACT_NCHW, false>(a, tm, tp, ks, s);
}
