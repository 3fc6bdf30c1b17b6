"""GPU parity of CHAIN on the 16-bit matrix cores (mb[1] = 3: every factor in two fp16 or three bf16 parts) at the sizes where it can go wrong:
odd numbers of k-groups in each contraction, channel counts and ranks that fill no block, tiles that leave part of a pixel
group or of the image empty, taps outside the image, the three ways x is read (NHWC, NCHW four bytes at a time, NCHW in aligned
runs of four pixels), every unit size."""
import numpy as np
import pytest

from parity_util import assert_parity, gpu_us
from paper_2211_03715_amd import binding as B
from paper_2211_03715_amd.workloads import Layer, make_inputs

pytestmark = pytest.mark.gpu

# (layer, tiles): the last three have 16 output pixels per compute unit and W % 4 == 0, so NCHW reads them in runs
CASES = [
    (Layer(2, 24, 40, 20, 18, 16, 24, 3, 1, 1), ((20, 18), (3, 5))),     # one z1 block: 9 k-groups, C = 1.5 groups of 16
    (Layer(3, 100, 148, 37, 28, 24, 40, 5, 1, 2), ((4, 8), (5, 7))),     # three z2 blocks, 5x5
    (Layer(2, 64, 64, 12, 16, 64, 80, 3, 2, 1), ((6, 8), (2, 4))),       # five z2 blocks, stride 2
    (Layer(1, 36, 36, 9, 7, 36, 52, 3, 1, 1), ((9, 7),)),                # three z1 blocks, four z2 blocks
    (Layer(1, 4, 4, 1, 1, 1, 1, 1, 1, 0), ((1, 1),)),                    # a single pixel
    (Layer(1, 12, 12, 15, 17, 6, 5, 7, 4, 6), ((2, 3), (6, 7))),         # 7x7, stride 4, taps far outside
    (Layer(40, 64, 96, 28, 28, 20, 33, 3, 2, 1), ((7, 14), (14, 12))),   # runs, stride 2
    (Layer(40, 20, 24, 12, 12, 16, 16, 3, 1, 1), ((12, 12), (5, 8))),    # runs, tiles past the last row and column
    (Layer(5, 8, 36, 32, 36, 50, 60, 1, 1, 0), ((4, 32), (8, 8))),       # runs, 1x1, C below one group
    # sums long enough for two fp16 parts, in runs: one and two z2 blocks (weights shared through LDS), five (not shared), C no
    # multiple of 32, tiles of five and more pixel blocks that end past the last row and column
    (Layer(40, 72, 24, 12, 12, 40, 16, 3, 1, 1), ((12, 12), (10, 8))),
    (Layer(40, 100, 36, 12, 12, 20, 32, 3, 1, 1), ((10, 8), (5, 12))),
    (Layer(40, 44, 24, 12, 12, 40, 80, 3, 1, 1), ((10, 8),)),
    (Layer(20, 104, 20, 32, 36, 24, 28, 3, 2, 1), ((10, 12),)),
]


def _run(layer, inputs, tuning, nhwc, bias=None, residual=None, offset=0, bf3=True, residual_offset=0):
    import torch
    from paper_2211_03715_amd.layer import TuckerConv2d
    dev = torch.device("cuda:0")
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a.transpose(0, 2, 3, 1) if nhwc else a)).to(dev)
    conv = TuckerConv2d(layer, 0, tuning, layout=B.LAYOUT_NHWC if nhwc else B.LAYOUT_NCHW)
    try:
        assert ("bf3" in conv.describe()) == bf3, conv.describe()
        fp16 = layer.C + layer.K ** 2 * layer.R1 + layer.R2 >= 208
        assert not bf3 or ("parts=fp16x2" if fp16 else "parts=bf16x3") in conv.describe(), conv.describe()
        w = [torch.from_numpy(inputs[k]).to(dev) for k in ("U_in", "core", "U_out")]
        conv.pack(*w)
        shape = conv.out_shape()
        whole = torch.full((offset + int(np.prod(shape)),), float("nan"), device=dev)
        y = whole[offset:].view(shape)                      # offset 1: only 4-byte aligned
        if residual is not None:
            beside = torch.zeros(residual_offset + residual.size, device=dev)
            beside[residual_offset:] = put(residual).flatten()
            residual = beside[residual_offset:].view(shape)
        conv(put(inputs["x"]), y, bias=None if bias is None else torch.from_numpy(bias).to(dev), residual=residual, relu=bias is not None)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        return got.transpose(0, 3, 1, 2) if nhwc else got
    finally:
        conv.close()


def _units(layer):
    nb1, nb2 = (layer.R1 + 15) // 16, (layer.R2 + 15) // 16
    return [(mb1, pb) for mb1 in (1, 2, 3) if mb1 <= nb1 for pb in ((2, 4) if nb2 <= 3 else (2,))]


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer,tiles", CASES, ids=lambda v: v.name() if isinstance(v, Layer) else "")
def test_chain3(orc, layer, tiles, nhwc):
    inputs = make_inputs(layer, 91)
    want, _ = orc.conv_factored(orc.Shape(**layer.asdict()), **inputs)
    rng = np.random.default_rng(6)
    bias = rng.standard_normal(layer.N, dtype=np.float32)
    residual = rng.standard_normal(want.shape, dtype=np.float32)
    with_epi = np.maximum(want + bias.astype(np.float64)[None, :, None, None] + residual, 0.0)
    for th, tw in tiles:
        for mb1, pb in _units(layer):
            t = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=th, tile_w=tw, waves=(4, 4, 4), mb=(mb1, 3, 1), pb=(pb,) * 3)
            print("[case] chain3", layer.name(), "nhwc" if nhwc else "nchw", th, tw, mb1, pb, flush=True)
            got = _run(layer, inputs, t, nhwc)
            assert_parity(got, want, "%s tile %dx%d units %d,%d" % (layer.name(), th, tw, mb1, pb))
            # three chained sums of at most 600 terms: fp32 multiply-adds show up to 1e-6, the split products no more; two
            # bf16 parts would show 5e-6 in each
            assert np.linalg.norm(got - want) <= 1.5e-6 * max(np.linalg.norm(want), 1e-30)
        # 16 bytes at a time where rows and tile allow it, then y and then the shortcut four bytes at a time
        for offset, r_offset in ((0, 0),) if nhwc else ((0, 0), (1, 0), (0, 1)):
            got = _run(layer, inputs, t, nhwc, bias, residual, offset, residual_offset=r_offset)
            assert_parity(got, with_epi, "%s tile %dx%d epilogue, y + %d floats, shortcut + %d" % (layer.name(), th, tw, offset, r_offset))


FLT_MAX = float(np.finfo(np.float32).max)


def _one_sign(a):
    return np.abs(a) + np.float32(1e-3)


# What reaches a sum that three bf16 parts cannot carry.  Gains below 1 keep the finite cases finite.
def _masked_x(i):                    # a mask value of the type's lowest
    i["x"][0, 3, 2:5, 3:9] = -FLT_MAX
    i["x"][-1, 1, 0, 0] = FLT_MAX


def _infinite_x(i):
    i["x"][0, 3, 4, 5], i["x"][-1, 2, 0, 0] = np.inf, -np.inf
    for k in ("U_in", "core", "U_out"):
        i[k][...] = _one_sign(i[k])


def _large_U_in(i):
    i["U_in"][2, 1] = FLT_MAX
    i["x"][...] *= np.float32(1e-20)


def _large_core(i):
    i["core"][3, 2, 0, 0] = -FLT_MAX
    i["x"][...] *= np.float32(1e-20)


def _large_U_out(i):
    i["U_out"][1, 4] = FLT_MAX
    i["x"][...] *= np.float32(1e-20)


def _infinite_core(i):
    i["x"][...], i["U_in"][...], i["U_out"][...] = _one_sign(i["x"]), _one_sign(i["U_in"]), _one_sign(i["U_out"])
    i["core"][2, 1, i["core"].shape[2] // 2, i["core"].shape[3] // 2] = np.inf


def _infinite_U_out(i):
    i["x"][...], i["U_in"][...], i["core"][...] = _one_sign(i["x"]), _one_sign(i["U_in"]), _one_sign(i["core"])
    i["U_out"][1, 2] = -np.inf


def _overflowing_z1(i):
    i["x"][0, :, 3, 3] = 1e30
    for k in ("U_in", "core", "U_out"):
        i[k][...] = _one_sign(i[k])
    i["U_in"][...] *= np.float32(1e12)


def _overflowing_y(i):
    for k in ("x", "U_in", "core", "U_out"):
        i[k][...] = _one_sign(i[k])
    i["x"][...] *= np.float32(1e18)
    i["U_out"][:, 2] *= np.float32(-1e30)


def _nan_x(i):
    i["x"][0, 3, 4, 5] = np.nan


def _nan_beside_infinity(i):
    _infinite_x(i)
    i["x"][0, 1, 1, 1] = np.nan


EXTREMES = (_masked_x, _infinite_x, _large_U_in, _large_core, _large_U_out, _infinite_core, _infinite_U_out, _overflowing_z1,
            _overflowing_y, _nan_x, _nan_beside_infinity)


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer,tiles", ((Layer(2, 32, 48, 12, 12, 32, 16, 3, 1, 1), ((12, 12), (4, 4))),
                                         (Layer(40, 20, 24, 12, 12, 16, 33, 3, 2, 1), ((6, 6), (5, 4))),
                                         (Layer(40, 20, 24, 12, 12, 40, 80, 1, 1, 0), ((12, 12), (5, 8))),
                                         # two fp16 parts, in runs: two z2 blocks, and four
                                         (Layer(40, 72, 24, 12, 12, 40, 20, 3, 1, 1), ((12, 12), (10, 8))),
                                         (Layer(80, 160, 24, 12, 12, 40, 60, 1, 1, 0), ((8, 12),))),
                         ids=lambda v: v.name() if isinstance(v, Layer) else "")
@pytest.mark.parametrize("extreme", EXTREMES, ids=lambda f: f.__name__[1:])
def test_values_without_three_parts_give_what_fp32_arithmetic_gives(orc, extreme, layer, tiles, nhwc):
    inputs = {k: v.copy() for k, v in make_inputs(layer, 92).items()}
    extreme(inputs)
    with np.errstate(invalid="ignore", over="ignore"):
        want = orc.conv_factored(orc.Shape(**layer.asdict()), **inputs)[0].astype(np.float32).astype(np.float64)
    for th, tw in tiles:
        fp32 = _run(layer, inputs, B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=th, tile_w=tw, waves=(4, 4, 4), mb=(1, 1, 1), pb=(1,) * 3), nhwc, bf3=False)
        t = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=th, tile_w=tw, waves=(4, 4, 4), mb=(1, 3, 1), pb=(2,) * 3)
        print("[case] chain3", extreme.__name__, layer.name(), "nhwc" if nhwc else "nchw", th, tw, flush=True)
        got = _run(layer, inputs, t, nhwc)
        # NaN, infinities and their signs exactly as the fp32 kernel has them; the rest as accurate as always, the outputs an
        # extreme value reaches and the others each against their own size
        assert np.array_equal(np.isnan(got), np.isnan(fp32)) and np.array_equal(np.where(np.isinf(got), got, 0), np.where(np.isinf(fp32), fp32, 0))
        finite = np.isfinite(got) & np.isfinite(want)
        assert extreme not in (_masked_x, _large_U_in, _large_core, _large_U_out) or np.isfinite(got).all()
        reached = np.abs(want) > (1e25 if extreme is _masked_x else 1e5)
        for part in (finite & reached, finite & ~reached):
            w, g = want[part], got.astype(np.float64)[part]
            assert part.sum() == 0 or np.linalg.norm(g - w) <= 1.5e-6 * max(np.linalg.norm(w), 1e-30)


SCALES = ((-116, 0, 0, 0), (0, -116, 0, 0), (0, 0, -116, 0), (0, 0, 0, -116), (-60, -56, 0, 0), (-50, 0, -66, 0), (-118, 60, 40, 0),
          (0, -60, -56, 100), (-113, 13, 0, 0))


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer,tile", ((Layer(2, 32, 48, 12, 12, 32, 16, 3, 1, 1), (4, 4)), (Layer(40, 20, 24, 12, 12, 40, 80, 3, 2, 1), (6, 6)),
                                        (Layer(40, 72, 24, 12, 12, 40, 20, 3, 1, 1), (10, 8))),
                         ids=lambda v: v.name() if isinstance(v, Layer) else "")
def test_the_scale_of_the_factors_costs_no_accuracy(orc, layer, tile, nhwc):
    """Factors, z1 or z2 below 2^-110 have no three bf16 parts with all their bits; nothing larger stands beside them here."""
    t = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=tile[0], tile_w=tile[1], waves=(4, 4, 4), mb=(2, 3, 1), pb=(2,) * 3)
    for scales in SCALES + ("part of the image",):
        inputs = {k: v.copy() for k, v in make_inputs(layer, 93).items()}
        small = np.zeros(inputs["x"].shape, bool)
        if isinstance(scales, str):
            small[0, :, 3:, :], small[1] = True, True
            inputs["x"][small] *= np.float32(2.0 ** -117)
        else:
            for k, e in zip(("x", "U_in", "core", "U_out"), scales):
                inputs[k] *= np.float32(2.0 ** e)
        want, _ = orc.conv_factored(orc.Shape(**layer.asdict()), **inputs)
        print("[case] chain3 scales", scales, layer.name(), "nhwc" if nhwc else "nchw", flush=True)
        got = _run(layer, inputs, t, nhwc).astype(np.float64)
        for part in (np.abs(want) < 1e-25, np.abs(want) >= 1e-25):
            assert not part.any() or np.linalg.norm((got - want)[part] * 2.0 ** 60) <= 1.5e-6 * np.linalg.norm(want[part] * 2.0 ** 60)


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer,tile", ((Layer(2, 72, 48, 12, 12, 32, 16, 3, 1, 1), (4, 4)), (Layer(40, 72, 24, 12, 12, 40, 80, 3, 2, 1), (6, 6))),
                         ids=lambda v: v.name() if isinstance(v, Layer) else "")
def test_values_far_from_those_that_set_the_scale(orc, layer, tile, nhwc):
    """x is scaled by the first 32 channels that a workgroup loads.  Channels behind them up to 512 times larger fit in fp16 and larger
    ones do not; pixels down to 2^-19 of them keep all their bits and smaller ones do not.  Both sides of each line."""
    t = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=tile[0], tile_w=tile[1], waves=(4, 4, 4), mb=(2, 3, 1), pb=(2,) * 3)
    for what, e in [("channels", e) for e in (4, 6, 7, 9, 11, 40)] + [("pixels", -e) for e in (10, 17, 19, 21, 23, 25, 40)]:
        inputs = {k: v.copy() for k, v in make_inputs(layer, 94).items()}
        if what == "channels":
            inputs["x"][:, -8:] *= np.float32(2.0 ** e)
        else:
            inputs["x"][0, :, 5:] *= np.float32(2.0 ** e)
        want, _ = orc.conv_factored(orc.Shape(**layer.asdict()), **inputs)
        print("[case] chain3, far from the scale", what, e, layer.name(), "nhwc" if nhwc else "nchw", flush=True)
        err = _run(layer, inputs, t, nhwc) - want
        # pixel by pixel, each against its own size: sums as in test_chain3
        assert (np.linalg.norm(err, axis=1) <= 1.5e-6 * np.linalg.norm(want, axis=1)).all()


def test_the_selector_takes_it_where_pixels_fill_the_chip():
    for lay in (B.LAYOUT_NCHW, B.LAYOUT_NHWC):
        t = B.tdc_select_tuning(B.make_shape(256, 128, 128, 28, 28, 32, 32, layout=lay))
        assert t.variant == B.VARIANT_CHAIN and t.mb[1] == 3 and t.tile_h * t.tile_w <= 128
        B.tdc_plan_destroy(B.tdc_plan_create(B.make_shape(256, 128, 128, 28, 28, 32, 32, layout=lay), 0, t))
        t = B.tdc_select_tuning(B.make_shape(32, 256, 256, 14, 14, 64, 64, layout=lay))
        assert t.mb[1] == 3 and t.tile_h * t.tile_w <= 32       # one group of pixel blocks that four wavefronts share
        assert B.tdc_select_tuning(B.make_shape(1, 256, 256, 14, 14, 64, 64, layout=lay)).variant != B.VARIANT_CHAIN
    # six z2 blocks: no such instance, the fp32 kernel takes the tuning
    t = B.make_tuning(variant=B.VARIANT_CHAIN, mb=(0, 3, 0))
    assert B.tdc_select_tuning(B.make_shape(64, 96, 96, 28, 28, 96, 96), tuning=t).mb[1] == 1


# the fp16 kernel (C + K*K*R1 + R2 >= 208): four bytes at a time, in runs with two and with four z2 blocks, NHWC; several channel groups
FP16_LAYERS = ((Layer(2, 72, 48, 12, 12, 32, 16, 3, 1, 1), (4, 4)), (Layer(40, 72, 24, 12, 12, 40, 20, 3, 1, 1), (12, 12)),
               (Layer(80, 160, 24, 12, 12, 40, 60, 1, 1, 0), (8, 12)))


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer,tile", FP16_LAYERS, ids=lambda v: v.name() if isinstance(v, Layer) else "")
def test_ranks_and_channels_that_the_next_factor_brings_to_one_size(orc, layer, tile, nhwc):
    """Rescaling x's channels, the ranks of U_in or those of the core and undoing it in the next factor leaves the layer what it
    is.  Also with pixels that use the smaller half only."""
    t = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=tile[0], tile_w=tile[1], waves=(4, 4, 4), mb=(1 if tile == (12, 12) else 2, 3, 1), pb=(2,) * 3)
    for bits in (8, 16, 20, 24, 28, 34, 40, 60):
        for what in ("channels", "ranks 1", "ranks 2", "half"):
            inputs = {k: v.copy() for k, v in make_inputs(layer, 95).items()}
            grade = lambda n: (2.0 ** np.round(np.linspace(bits, 0, n))).astype(np.float32)
            if what == "channels":
                s = grade(layer.C)
                inputs["x"] *= s[None, :, None, None]
                inputs["U_in"] /= s[:, None]
            elif what == "ranks 2":
                s = grade(layer.R2)
                inputs["core"] *= s[None, :, None, None]
                inputs["U_out"] /= s[:, None]
            else:
                s = grade(layer.R1)
                if what == "half":                       # the first half of the channels feeds the first, larger, half of the ranks
                    s[:layer.R1 // 2], s[layer.R1 // 2:] = 2.0 ** bits, 1
                    inputs["U_in"][:layer.C // 2, layer.R1 // 2:] = 0
                    inputs["U_in"][layer.C // 2:, :layer.R1 // 2] = 0
                    inputs["x"][0, :layer.C // 2, :, 5:] = 0
                inputs["U_in"] *= s[None, :]
                inputs["core"] /= s[:, None, None, None]
            want, _ = orc.conv_factored(orc.Shape(**layer.asdict()), **inputs)
            print("[case] chain3,", what, "2^%d apart" % bits, layer.name(), "nhwc" if nhwc else "nchw", flush=True)
            err = _run(layer, inputs, t, nhwc) - want
            assert (np.linalg.norm(err, axis=1) <= 1.5e-6 * np.linalg.norm(want, axis=1)).all(), (what, bits)


def _larger_late(i):                 # behind what sets the scale
    i["x"][:, -8:] *= np.float32(200.0)


def _flat(i):                        # sums without a change of sign, C times a product and not sqrt(C)
    i["x"][...] = 1.9
    i["U_in"][...] = 0.05


def _dead(i):                        # filters without a weight, images without a value
    i["U_out"][:, ::2] = 0
    i["U_out"][:, :17] = 0
    i["x"][1::2] = 0


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer,tile", ((Layer(32, 512, 64, 14, 14, 32, 32, 3, 1, 1), (4, 14)), (Layer(32, 256, 128, 14, 14, 64, 64, 3, 1, 1), (2, 14))),
                         ids=lambda v: v.name() if isinstance(v, Layer) else "")
@pytest.mark.parametrize("values", (_larger_late, _flat, _dead), ids=lambda f: f.__name__[1:])
def test_finite_inputs_that_fp16_holds_cost_the_usual_time(values, layer, tile, nhwc):
    """They are not computed again in fp32, which takes several times as long."""
    import torch
    from paper_2211_03715_amd.layer import TuckerConv2d
    dev = torch.device("cuda:0")
    usual = make_inputs(layer, 96)
    other = {k: v.copy() for k, v in usual.items()}
    values(other)
    t = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=tile[0], tile_w=tile[1], waves=(4, 4, 4), mb=(2, 3, 1), pb=(2,) * 3)
    us = []
    for inputs in (usual, other):
        conv = TuckerConv2d(layer, 0, t, B.LAYOUT_NHWC if nhwc else B.LAYOUT_NCHW)
        try:
            w = [torch.from_numpy(inputs[k]).to(dev) for k in ("U_in", "core", "U_out")]
            conv.pack(*w)
            x = torch.from_numpy(np.ascontiguousarray(inputs["x"].transpose(0, 2, 3, 1) if nhwc else inputs["x"])).to(dev)
            y = torch.empty(conv.out_shape(), device=dev)
            launch = conv.bind(x, y)
            gpu_us(launch)
            us.append(gpu_us(launch))
            if values is _dead and inputs is other:
                got = y.permute(0, 3, 1, 2) if nhwc else y
                assert not got[:, ::2].any() and not got[:, :17].any() and not got[1::2].any() and got[0, 17].any()
        finally:
            conv.close()
    print("[case] chain3,", values.__name__, layer.name(), "nhwc" if nhwc else "nchw", "%.1f us, usually %.1f" % (us[1], us[0]), flush=True)
    assert us[1] <= 1.5 * us[0]


def test_a_plan_takes_no_lds_for_weights_that_its_kernel_does_not_share():
    """Instances that read runs and hold three or more z2 blocks keep z1 only: 9 x 57 pixels in 33 blocks, two channel blocks of
    64 bytes a pixel, and 32 bytes.  The others keep two chunks of weights beside it."""
    layer = Layer(32, 128, 256, 56, 56, 32, 64, 3, 2, 1)
    for lay, extra in ((B.LAYOUT_NCHW, 0), (B.LAYOUT_NHWC, 2 * 8 * 1024)):
        t = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=4, tile_w=28, waves=(4, 4, 4), mb=(2, 3, 1), pb=(2,) * 3)
        plan = B.tdc_plan_create(B.make_shape(*[getattr(layer, k) for k in ("batch", "C", "N", "H", "W", "R1", "R2", "K", "stride", "pad")], layout=lay), 0, t)
        try:
            assert "lds=%dB" % (32 + 64 * 2 * 16 * 33 + extra) in B.tdc_plan_describe(plan)
        finally:
            B.tdc_plan_destroy(plan)


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer,tile", ((Layer(64, 128, 128, 28, 28, 32, 32, 3, 1, 1), (4, 28)), (Layer(32, 256, 256, 14, 14, 64, 64, 3, 1, 1), (2, 14))),
                         ids=lambda v: v.name() if isinstance(v, Layer) else "")
def test_nan_inputs_cost_a_second_pass_at_most(layer, tile, nhwc):
    """Every value NaN, or one pixel in 64: the outputs they reach are NaN without being computed again, the others keep theirs.
    Finding that out reads x once more, unpipelined: 1.5 to 2.5 times the usual time, 4 allowed; the tiles in fp32 would be 4 to 5."""
    import torch
    from paper_2211_03715_amd.layer import TuckerConv2d
    dev = torch.device("cuda:0")
    inputs = make_inputs(layer, 97)
    x = torch.from_numpy(np.ascontiguousarray(inputs["x"].transpose(0, 2, 3, 1) if nhwc else inputs["x"])).to(dev)
    some = x.clone()
    (some[:, ::8, ::8, 5] if nhwc else some[:, 5, ::8, ::8]).fill_(float("nan"))
    t = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=tile[0], tile_w=tile[1], waves=(4, 4, 4), mb=(2, 3, 1), pb=(2,) * 3)
    conv = TuckerConv2d(layer, 0, t, B.LAYOUT_NHWC if nhwc else B.LAYOUT_NCHW)
    try:
        w = [torch.from_numpy(inputs[k]).to(dev) for k in ("U_in", "core", "U_out")]
        conv.pack(*w)
        y = torch.empty(conv.out_shape(), device=dev)
        gpu_us(conv.bind(x, y))
        usual, clean = gpu_us(conv.bind(x, y)), y.clone()
        for what, bad in (("every value", torch.full_like(x, float("nan"))), ("some pixels", some)):
            took = gpu_us(conv.bind(bad, y))
            print("[case] chain3, NaN in", what, layer.name(), "nhwc" if nhwc else "nchw", "%.1f us, usually %.1f" % (took, usual), flush=True)
            assert took <= 4 * usual
            nan = torch.isnan(y)
            assert nan.all() if bad is not some else nan.any()
            assert bad is not some or (y[~nan] - clean[~nan]).norm() <= 1e-6 * clean[~nan].norm()
    finally:
        conv.close()


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer,tile", FP16_LAYERS, ids=lambda v: v.name() if isinstance(v, Layer) else "")
@pytest.mark.parametrize("what", ("beyond_fp16", "late_channels", "overflowing_z1", "wide_weights", "infinite_weight", "nan_weight", "alone"))
def test_a_nan_explains_no_outputs_but_its_own(orc, what, layer, tile, nhwc):
    """One NaN beside finite values that fp16 does not hold at the scale the workgroup takes, beside z1 that it does not hold, and with weights
    that are kept out of the parts or are no numbers."""
    inputs = {k: v.copy() for k, v in make_inputs(layer, 98).items()}
    if what == "beyond_fp16":
        inputs["x"][0, :, 0, 3:6] *= np.float32(2.0 ** 14)
    elif what == "late_channels":
        inputs["x"][:, -8:] *= np.float32(2.0 ** 14)
    elif what == "overflowing_z1":
        inputs["x"][0, :, 2:4, 3:5] = 300.0
        inputs["U_in"][...] = 1.0
        for k in ("core", "U_out"):                      # z1's channels are all alike: no differences of theirs
            inputs[k] = np.abs(inputs[k])
    elif what == "wide_weights":
        inputs["U_out"][:2, 7] = 2.0 ** 12, 2.0 ** -20
    elif what == "infinite_weight":
        inputs["U_out"][1, 2] = np.inf
    elif what == "nan_weight":
        inputs["U_out"][1, 2] = np.nan
    inputs["x"][0, 3, 0, 0] = np.nan
    t = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=tile[0], tile_w=tile[1], waves=(4, 4, 4), mb=(1 if tile == (12, 12) else 2, 3, 1), pb=(2,) * 3)
    with np.errstate(invalid="ignore", over="ignore"):
        want, _ = orc.conv_factored(orc.Shape(**layer.asdict()), **inputs)
    print("[case] chain3, one NaN,", what, layer.name(), "nhwc" if nhwc else "nchw", flush=True)
    got = _run(layer, inputs, t, nhwc)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    with np.errstate(invalid="ignore"):
        err, ref = np.where(np.isfinite(want), got - want, 0), np.where(np.isfinite(want), want, 0)
    assert (np.linalg.norm(err, axis=(2, 3)) <= 1.5e-6 * np.linalg.norm(ref, axis=(2, 3))).all()      # an image's channel


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("tile,at", (((5, 7), (5, 0)), ((5, 7), (25, 7)), ((2, 14), (2, 0)), ((6, 28), (6, 0))))
def test_one_output_that_is_small_by_chance_has_no_tile_computed_again(orc, tile, at, nhwc):
    """A channel that the first pixel of a tile's z2 happens to give nothing: in the tile's last blocks, which the tile does not fill, that
    pixel stands in for those past the last; in the tiles that end two rows past the image it is all that they hold.  The other channels would not keep their bits if the tile were computed again."""
    layer = Layer(2, 128, 128, 28, 28, 32, 32, 3, 1, 1)
    inputs = {k: v.copy() for k, v in make_inputs(layer, 99).items()}
    z2, _ = orc.conv_factored(orc.Shape(**dict(layer.asdict(), batch=1, N=layer.R2)), inputs["x"][:1], inputs["U_in"], inputs["core"], np.eye(layer.R2, dtype=np.float32))
    t = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=tile[0], tile_w=tile[1], waves=(4, 4, 4), mb=(2, 3, 1), pb=(2,) * 3)
    clean = _run(layer, inputs, t, nhwc)
    z = z2[0, :, at[0], at[1]].astype(np.float64)
    u = inputs["U_out"][:, 7].astype(np.float64)
    inputs["U_out"][:, 7] = u - z * (z @ u) / (z @ z)
    print("[case] chain3, small by chance", tile, at, "nhwc" if nhwc else "nchw", flush=True)
    got = _run(layer, inputs, t, nhwc)
    others = np.arange(layer.N) != 7
    assert abs(got[0, 7, at[0], at[1]]) < 1e-5 and np.array_equal(got[:, others], clean[:, others])
