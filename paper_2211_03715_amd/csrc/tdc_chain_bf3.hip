// CHAIN on the bf16 matrix cores, host side: the launch.  Which layers take it and its tile geometry are in tdc_chain3.hip, the
// kernel is in tdc_chain_bf3_kernel.h; its instances are compiled in tdc_chain_bf3_nchw.hip, tdc_chain_bf3_runs.hip and
// tdc_chain_bf3_nhwc.hip.
#include "tdc_chain_bf3_kernel.h"

hipError_t tdc_launch_chain_bf3_nchw(const TdcChainBf3Args &, int, int, int, dim3, size_t, hipStream_t, bool);
hipError_t tdc_launch_chain_bf3_runs(const TdcChainBf3Args &, int, int, int, dim3, size_t, hipStream_t, bool);
hipError_t tdc_launch_chain_bf3_nhwc(const TdcChainBf3Args &, int, int, int, dim3, size_t, hipStream_t, bool);

hipError_t tdc_launch_chain_bf3(const TdcDims &d, const tdc_tuning &t, const TdcFusedGeom &g, hipStream_t s, const float *x,
                                const void *uin_p3, const void *core_p3, const void *uout_p3, float *y, const TdcEpi &epi, bool prepare_only)
{
    TdcChainBf3Args a;
    a.x = x; a.uin3 = uin_p3; a.core3 = core_p3; a.uout3 = uout_p3; a.y = y; a.epi = epi;
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
    // rows of whole quads and a 16-byte aligned y; otherwise the same values go out as four 4-byte stores
    a.vec = g.TW % 4 == 0 && d.Wo % 4 == 0 && ((uintptr_t)y & 15u) == 0;
    a.uin_bytes = (unsigned)tdc_packed3_bytes(d.NB1, d.KG1);
    a.core_bytes = (unsigned)tdc_packed3_bytes(d.NB2, a.KG2);
    a.uout_bytes = (unsigned)tdc_packed3_bytes(d.NB3, d.NB2);
    a.div_tiles_x = tdc_make_div((unsigned)g.tiles_x); a.div_tiles = tdc_make_div((unsigned)a.tiles);
    a.div_QW = tdc_make_div((unsigned)g.QW); a.div_TW = tdc_make_div((unsigned)g.TW);
    a.div_NB1 = tdc_make_div((unsigned)d.NB1); a.div_K = tdc_make_div((unsigned)d.K);
    a.div_RPR = tdc_make_div((unsigned)a.RPR); a.div_mg1 = tdc_make_div((unsigned)a.n_mg1);
    const dim3 grid((unsigned)a.tiles, (unsigned)d.B);
    const auto launch = lay == TDC_LAY_NHWC ? tdc_launch_chain_bf3_nhwc : lay == TDC_LAY_NCHW_RUNS ? tdc_launch_chain_bf3_runs : tdc_launch_chain_bf3_nchw;
    return launch(a, d.NB2, t.pb[0], t.mb[0], grid, g.lds_bytes, s, prepare_only);
}
