// CHAIN on the fp16 matrix cores, host side: which shapes it covers, its tile geometry, and the launch.  The kernel is in
// tdc_chain3_kernel.h; its instances are compiled in tdc_chain3_nchw.hip, tdc_chain3_runs.hip and tdc_chain3_nhwc.hip.
#include <algorithm>
#include <cmath>

#include "tdc_chain3_kernel.h"

hipError_t tdc_launch_chain3_nchw(const TdcChain3Args &, int, int, int, dim3, size_t, hipStream_t, bool);
hipError_t tdc_launch_chain3_runs(const TdcChain3Args &, int, int, int, dim3, size_t, hipStream_t, bool);
hipError_t tdc_launch_chain3_nhwc(const TdcChain3Args &, int, int, int, dim3, size_t, hipStream_t, bool);

bool tdc_chain3_supported(const TdcDims &d, int mb1, int pb)
{
    if (mb1 < 1 || mb1 > 3 || mb1 > d.NB1) return false;
    // every weight array lies behind one buffer descriptor
    const size_t lim = 1ull << 31;
    if (tdc_packed3_bytes(d.NB1, d.KG1) >= lim || tdc_packed3_bytes(d.NB2, d.K * d.K * d.NB1) >= lim || tdc_packed3_bytes(d.NB3, d.NB2) >= lim) return false;
#define TDC_X(N_, P_) if (d.NB2 == N_ && pb == P_) return true;
    TDC_CHAIN3_UNITS(TDC_X)
#undef TDC_X
    return false;
}

int tdc_chain3_share(int pixel_groups) { return pixel_groups == 1 ? 2 : pixel_groups == 2 ? 1 : 0; }

TdcFusedGeom tdc_chain3_geometry(const TdcDims &d, int tile_h, int tile_w, int pb)
{
    TdcFusedGeom g;
    g.TH = tile_h;
    g.TW = tile_w;
    g.QH = (tile_h - 1) * d.stride + d.K;
    g.QW = (tile_w - 1) * d.stride + d.K;
    g.Q = g.QH * g.QW;
    g.QB = (g.Q + 15) / 16;
    g.PBk = (tile_h * tile_w + 15) / 16;
    g.tiles_x = (d.Wo + tile_w - 1) / tile_w;
    g.tiles_y = (d.Ho + tile_h - 1) / tile_h;
    g.pitch1 = 16 * (g.QB | 1);       // an odd number of 128-byte rows: lane groups 2i and 2i + 1 use different halves of the banks
    g.pitch2 = 0;
    g.weights_in_lds = g.weights_fit = false;
    const bool bf3 = tdc_chain3_bf3(d);
    g.lds_bytes = bf3 ? (size_t)96 * d.NB1 * g.pitch1 : sizeof(Chain3Shared) + (size_t)64 * d.NB1 * g.pitch1;
    if (pb <= 0) return g;
    const int lay = d.nhwc ? TDC_LAY_NHWC : d.s1_runs ? TDC_LAY_NCHW_RUNS : TDC_LAY_NCHW;
    if (tdc_chain3_share((g.PBk + pb - 1) / pb)) g.lds_bytes += (size_t)TDC_CHAIN3_WAVES * d.NB2 * pb * 1024;
    else if (!bf3 && chain3_shares_weights(lay, d.NB2)) g.lds_bytes += (size_t)2048 * chain3_feed_pieces(d.NB2);
    return g;
}

hipError_t tdc_launch_chain3(const TdcDims &d, const tdc_tuning &t, const TdcFusedGeom &g, hipStream_t s, const float *x,
                             const void *uin_sp, const void *core_sp, const void *uout_sp, float *y, const TdcEpi &epi, bool prepare_only)
{
    if (tdc_chain3_bf3(d)) return tdc_launch_chain_bf3(d, t, g, s, x, uin_sp, core_sp, uout_sp, y, epi, prepare_only);
    TdcChain3Args a;
    a.x = x; a.uin = uin_sp; a.core = core_sp; a.uout = uout_sp; a.y = y; a.epi = epi;
    a.C = d.C; a.N = d.N; a.H = d.H; a.W = d.W; a.Ho = d.Ho; a.Wo = d.Wo; a.K = d.K; a.stride = d.stride; a.pad = d.pad;
    a.NB1 = d.NB1; a.NB3 = d.NB3; a.S1 = (d.KG1 + 1) / 2; a.KG2 = d.K * d.K * d.NB1; a.S2 = (a.KG2 + 1) / 2;
    a.TH = g.TH; a.TW = g.TW; a.QH = g.QH; a.QW = g.QW; a.Q = g.Q; a.P = g.TH * g.TW; a.QB = g.QB;
    a.n_pg2 = (g.PBk + t.pb[0] - 1) / t.pb[0];
    a.lg_ks = tdc_chain3_share(a.n_pg2);
    a.pitch1 = g.pitch1;
    const int lay = d.nhwc ? TDC_LAY_NHWC : d.s1_runs ? TDC_LAY_NCHW_RUNS : TDC_LAY_NCHW;
    a.RPR = tdc_runs_per_row(d.W, d.Wo, g.TW, d.K, d.stride, d.pad);
    a.n_pg1 = lay == TDC_LAY_NCHW_RUNS ? (g.QH * a.RPR + 15) / 16 : (g.QB + 1) / 2;
    a.n_mg1 = (d.NB1 + t.mb[0] - 1) / t.mb[0];
    a.tiles_x = g.tiles_x; a.tiles = g.tiles_x * g.tiles_y;
    a.xcd_per = (int)((long)a.tiles * d.B / 8); a.xcd_rem = (int)((long)a.tiles * d.B % 8);
    // rows of whole quads, y and shortcut 16-byte aligned; otherwise the same values go out, and come in, four bytes at a time
    a.vec = g.TW % 4 == 0 && d.Wo % 4 == 0 && (((uintptr_t)y | (uintptr_t)epi.residual) & 15u) == 0;
    a.uin_bytes = (unsigned)tdc_split_bytes(2, d.NB1, d.KG1);
    a.core_bytes = (unsigned)tdc_split_bytes(2, d.NB2, a.KG2);
    a.uout_bytes = (unsigned)tdc_split_bytes(2, d.NB3, d.NB2);
    // Scaled weights of 2^12 and x of 2^4.5 give sums of sqrt(C) 2^16.5; where neither changes sign they reach C 2^20, still below 2^16
    // at 4096 channels.
    a.z1_exp = 11 + (int)std::lround(0.5 * std::log2((double)d.C));
    // A channel's largest output among a lane's pixels must be 2^22 times what the parts lose.  With scaled weights of 2^12 and values of
    // 2^12 at most, root mean square, z1 is off by 2^-36 (x, U_in and its own parts), the scaled z2 by sqrt(K K R1) 2^-23.5 before its
    // scale 2^z2_exp and by its parts' 2^-37 behind it, and the sums of the outputs by sqrt(R2) (2^12 of that + 2^-25).  Normal values
    // give 2^17 times more.  As exponents: of what comes from in front of z2's scale, with that 0, and of the rest.
    const double r2 = 0.5 * std::log2((double)d.R2);
    a.lost2 = (int)std::lround(11 + r2 + 0.5 * std::log2((double)d.K * d.K * d.R1));
    a.lost3 = (int)std::lround(r2 - 2);
    a.div_tiles_x = tdc_make_div((unsigned)g.tiles_x); a.div_tiles = tdc_make_div((unsigned)a.tiles);
    a.div_QW = tdc_make_div((unsigned)g.QW); a.div_TW = tdc_make_div((unsigned)g.TW);
    a.div_NB1 = tdc_make_div((unsigned)d.NB1); a.div_K = tdc_make_div((unsigned)d.K);
    a.div_RPR = tdc_make_div((unsigned)a.RPR); a.div_mg1 = tdc_make_div((unsigned)a.n_mg1);
    const dim3 grid((unsigned)a.tiles, (unsigned)d.B);
    const auto launch = lay == TDC_LAY_NHWC ? tdc_launch_chain3_nhwc : lay == TDC_LAY_NCHW_RUNS ? tdc_launch_chain3_runs : tdc_launch_chain3_nchw;
    return launch(a, d.NB2, t.pb[0], t.mb[0], grid, g.lds_bytes, s, prepare_only);
}
