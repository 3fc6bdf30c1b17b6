"""GPU parity of the dense layer in tiles on the 16-bit matrix cores (every factor in two or three parts), at the sizes where its
tiling can go wrong: contractions that are not whole steps (two 16-wide k-groups), channel counts and pixel counts that leave
part of a tile empty, images much smaller than a tile, taps outside the image, both activation layouts, both tile heights,
the contraction dealt to one and to two groups of wavefronts."""
import numpy as np
import pytest

from parity_util import assert_parity, gpu_us
from paper_2211_03715_amd import binding as B
from paper_2211_03715_amd.workloads import Layer, make_dense_inputs

pytestmark = pytest.mark.gpu

LAYERS = [
    Layer(1, 16, 64, 8, 8, 1, 1, 1, 1, 0),         # one k-group: half a step, one exact tile
    Layer(1, 32, 128, 8, 8, 1, 1, 1, 1, 0),        # one step
    Layer(70, 48, 68, 1, 1, 1, 1, 1, 1, 0),        # single-pixel images, 1.5 steps, pixels and channels just past a tile
    Layer(9, 100, 60, 3, 5, 1, 1, 1, 1, 0),        # several images per tile, C no multiple of 16, N below a tile
    Layer(2, 64, 132, 13, 9, 1, 1, 1, 2, 0),       # strided 1x1 (a projection shortcut)
    Layer(3, 20, 24, 19, 23, 1, 1, 3, 1, 1),       # K x K, 4.5 steps of which none holds one tap alone
    Layer(2, 36, 72, 16, 12, 1, 1, 3, 2, 1),
    Layer(1, 12, 8, 7, 40, 1, 1, 5, 1, 2),
    Layer(2, 8, 16, 9, 8, 1, 1, 7, 3, 6),          # taps far outside, stride 3
]


def _oracle(orc, layer, inputs, bias=None, residual=None):
    want, _ = orc.conv_dense_with(orc.Shape(**layer.asdict()), inputs["x"], inputs["W"].astype(np.float64))
    if bias is not None:
        want = np.maximum(want + bias.astype(np.float64)[None, :, None, None] + residual, 0.0)
    return want


def _run(layer, inputs, tm, waves, nhwc, bias=None, residual=None, offset=0, in_lds=None, parts=""):
    import torch
    from paper_2211_03715_amd.layer import DenseConv2d
    dev = torch.device("cuda:0")
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a.transpose(0, 2, 3, 1) if nhwc else a)).to(dev)
    conv = DenseConv2d(layer, 0, B.make_tuning(tile_h=tm, tile_w=64, waves=(waves,) * 3), B.LAYOUT_NHWC if nhwc else B.LAYOUT_NCHW)
    try:
        assert in_lds is None or ("pixels-in-lds" in conv.describe()) == in_lds, conv.describe()
        assert not parts or "parts=" + parts in conv.describe(), conv.describe()
        W = torch.from_numpy(inputs["W"]).to(dev)
        conv.pack(W)
        shape = conv.out_shape()
        whole = torch.full((offset + int(np.prod(shape)),), float("nan"), device=dev)
        y = whole[offset:].view(shape)                      # offset 1: only 4-byte aligned
        conv(put(inputs["x"]), y, bias=None if bias is None else torch.from_numpy(bias).to(dev),
             residual=None if residual is None else put(residual), relu=bias is not None)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        return got.transpose(0, 3, 1, 2) if nhwc else got
    finally:
        conv.close()


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer", LAYERS, ids=lambda l: l.name())
def test_tiles(orc, layer, nhwc):
    if nhwc and (layer.C % 4 or layer.N % 4):
        pytest.skip("NHWC needs channel counts that are multiples of 4")
    inputs = make_dense_inputs(layer, 77)
    want = _oracle(orc, layer, inputs)
    for tm in (64, 128):
        for waves in (4, 8):
            print("[case] tiles", layer.name(), "nhwc" if nhwc else "nchw", tm, waves, flush=True)
            got = _run(layer, inputs, tm, waves, nhwc)
            assert_parity(got, want, "%s tile %d waves %d" % (layer.name(), tm, waves))
            # fp32 sums of at most 800 terms here: an fp32 chain shows about 6e-7 (sqrt(800) roundings of 2^-25 relative to the
            # root of the sum), the split products about the same; two bf16 parts would show 5e-6
            rel = np.linalg.norm(got - want) / np.linalg.norm(want)
            assert rel <= 1.2e-6, rel


@pytest.mark.parametrize("nhwc,offset", ((False, 0), (False, 1), (True, 0)), ids=("nchw", "nchw_4_byte_aligned_y", "nhwc"))
def test_tiles_with_epilogue(orc, nhwc, offset):
    """Bias, shortcut and ReLU in the store; P = 12 (16-byte stores in NCHW) and P = 15 (quads that cross an image)."""
    for layer in (Layer(7, 40, 72, 3, 4, 1, 1, 1, 1, 0), Layer(7, 40, 72, 3, 5, 1, 1, 1, 1, 0)):
        print("[case] tiles epilogue", layer.name(), nhwc, offset, flush=True)
        inputs = make_dense_inputs(layer, 78)
        rng = np.random.default_rng(5)
        bias = rng.standard_normal(layer.N, dtype=np.float32)
        residual = rng.standard_normal((layer.batch, layer.N, layer.Ho, layer.Wo), dtype=np.float32)
        got = _run(layer, inputs, 64, 4, nhwc, bias, residual, offset)
        assert_parity(got, _oracle(orc, layer, inputs, bias, residual), layer.name())


def test_the_selector_takes_tiles_for_large_launches_only():
    """A batch of 32 goes to the tiles, the same layer at batch 1 does not, and a chosen tile is accepted when forced."""
    for lay in (B.LAYOUT_NCHW, B.LAYOUT_NHWC):
        dense = B.make_tuning(variant=B.VARIANT_DENSE)
        assert B.tdc_select_tuning(B.make_shape(1, 1024, 256, 14, 14, 1, 1, 1, 1, 0, lay), tuning=dense).as_dict()["tile_h"] == 0
        shape = B.make_shape(32, 1024, 256, 14, 14, 1, 1, 1, 1, 0, lay)
        t = B.tdc_select_tuning(shape, tuning=B.make_tuning(variant=B.VARIANT_DENSE))
        assert t.as_dict()["tile_h"] in (64, 128) and t.as_dict()["tile_w"] == 64
        B.tdc_plan_destroy(B.tdc_plan_create(shape, 0, t))
    for bad in (dict(tile_h=96, tile_w=64), dict(tile_h=64, tile_w=128), dict(tile_h=64, tile_w=64, waves=(3, 3, 3))):
        with pytest.raises(B.TdcError):
            B.tdc_plan_create(B.make_shape(1, 64, 64, 8, 8, 1, 1, 1, 1, 0), 0, B.make_tuning(variant=B.VARIANT_DENSE, **bad))


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer", (Layer(2, 40, 72, 13, 9, 1, 1, 3, 1, 1), Layer(2, 40, 72, 8, 8, 1, 1, 1, 1, 0)), ids=lambda l: l.name())
def test_infinite_inputs_give_what_fp32_arithmetic_gives(orc, layer, nhwc):
    """An infinite value has no three parts; the outputs it reaches are infinities of the right sign all the same, and those it
    does not reach keep their accuracy."""
    inputs = make_dense_inputs(layer, 79)
    inputs["x"][0, 3, 4, 5] = np.inf
    with np.errstate(invalid="ignore"):
        want = _oracle(orc, layer, inputs)
    for tm, waves in ((64, 4), (128, 8)):
        print("[case] tiles, infinite input", layer.name(), "nhwc" if nhwc else "nchw", tm, waves, flush=True)
        got = _run(layer, inputs, tm, waves, nhwc)
        finite = np.isfinite(want)
        assert (~finite).any() and np.array_equal(got[~finite], want[~finite].astype(np.float32))
        assert_parity(got[finite], want[finite], layer.name())


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer", (Layer(2, 24, 72, 13, 9, 1, 1, 3, 1, 1), Layer(2, 72, 72, 8, 8, 1, 1, 1, 1, 0)), ids=lambda l: l.name())
@pytest.mark.parametrize("value", (np.finfo(np.float32).max, 3.4e38, np.inf), ids=("largest", "just_above_bf16", "infinite"))
def test_weights_without_three_parts_give_what_fp32_arithmetic_gives(orc, value, layer, nhwc):
    """The largest finite weights round to infinity in bf16.  9 and 3 steps: the second of two groups of wavefronts multiplies a
    step past the end.  With the epilogue, whose ReLU would make a NaN a 0."""
    inputs = make_dense_inputs(layer, 80)
    inputs["W"][5, 7, layer.K // 2, layer.K // 2] = value
    inputs["x"] = np.abs(inputs["x"]) * np.float32(1e-12)
    rng = np.random.default_rng(6)
    bias = rng.standard_normal(layer.N, dtype=np.float32)
    residual = rng.standard_normal((layer.batch, layer.N, layer.Ho, layer.Wo), dtype=np.float32)
    want = _oracle(orc, layer, inputs, bias, residual)
    for tm, waves in ((64, 4), (128, 8)):
        print("[case] tiles, weight", value, layer.name(), "nhwc" if nhwc else "nchw", tm, waves, flush=True)
        got = _run(layer, inputs, tm, waves, nhwc, bias, residual)
        reached = np.zeros(want.shape, bool)
        reached[:, 7] = True
        if np.isinf(value):
            assert np.array_equal(got[reached], want[reached].astype(np.float32))
        else:
            assert_parity(got[reached], want[reached], layer.name())
        assert_parity(got[~reached], want[~reached], layer.name())


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
def test_an_infinite_weight_at_taps_outside_the_image_is_no_part_of_the_sum(orc, nhwc):
    layer = Layer(2, 24, 72, 13, 9, 1, 1, 3, 1, 1)
    inputs = make_dense_inputs(layer, 81)
    inputs["x"], inputs["W"][4, 9, 0, 2] = np.abs(inputs["x"]), -np.inf
    inputs["x"][1, 3, 6, 6] = np.nan
    want = _oracle(orc, layer, inputs)
    for tm, waves in ((64, 4), (128, 8)):
        print("[case] tiles, infinite weight", "nhwc" if nhwc else "nchw", tm, waves, flush=True)
        got = _run(layer, inputs, tm, waves, nhwc)
        finite = np.isfinite(want)
        assert np.array_equal(got[~finite], want[~finite].astype(np.float32), equal_nan=True) and np.isinf(want).any() and np.isnan(want).any()
        assert_parity(got[finite], want[finite], layer.name())


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer", (Layer(8, 128, 128, 28, 28, 1, 1, 3, 1, 1), Layer(8, 512, 128, 28, 28, 1, 1, 1, 1, 0)), ids=lambda l: l.name())
def test_nan_inputs_cost_a_second_pass_at_most(layer, nhwc):
    """Every value NaN, or one pixel in 64: the sums they reach are NaN without being computed again, the others keep theirs.
    Finding that out reads the factors once more, unpipelined: 2 to 3 times the usual time, 6 allowed; computing the
    outputs one after the other would be 100 times."""
    import torch
    from paper_2211_03715_amd.layer import DenseConv2d
    dev = torch.device("cuda:0")
    inputs = make_dense_inputs(layer, 82)
    x = torch.from_numpy(np.ascontiguousarray(inputs["x"].transpose(0, 2, 3, 1) if nhwc else inputs["x"])).to(dev)
    some = x.clone()
    (some[:, ::8, ::8, 5] if nhwc else some[:, 5, ::8, ::8]).fill_(float("nan"))
    conv = DenseConv2d(layer, 0, B.make_tuning(tile_h=64, tile_w=64, waves=(4,) * 3), B.LAYOUT_NHWC if nhwc else B.LAYOUT_NCHW)
    try:
        W = torch.from_numpy(inputs["W"]).to(dev)
        conv.pack(W)
        y = torch.empty(conv.out_shape(), device=dev)

        def us(inp):
            launch, best = conv.bind(inp, y), 1e9
            for _ in range(5):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                for _ in range(10):
                    launch()
                b.record()
                b.synchronize()
                best = min(best, a.elapsed_time(b) * 100)
            return best

        us(x)
        usual, clean = us(x), y.clone()
        for what, bad in (("every value", torch.full_like(x, float("nan"))), ("some pixels", some)):
            took = us(bad)
            print("[case] tiles, NaN in", what, layer.name(), "nhwc" if nhwc else "nchw", "%.1f us, usually %.1f" % (took, usual), flush=True)
            assert took <= 6 * usual
            nan = torch.isnan(y)
            assert nan.all() if bad is not some else (nan.any() and torch.equal(y[~nan], clean[~nan]))
    finally:
        conv.close()


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer", (Layer(2, 40, 72, 13, 9, 1, 1, 3, 1, 1), Layer(2, 40, 72, 8, 8, 1, 1, 1, 1, 0)), ids=lambda l: l.name())
def test_the_scale_of_the_factors_costs_no_accuracy(orc, layer, nhwc):
    """Factors below 2^-110 have no three bf16 parts with all their bits.  Whole tensors, a few pixels, and a few filters (whose
    outputs keep the accuracy that weights of 2^-100 allow)."""
    for what in ((-116, 0), (0, -116), (-60, -56), (-119, 60), (-113, 13), "pixels", "filters"):
        inputs = make_dense_inputs(layer, 83)
        if what == "pixels":
            inputs["x"][0, :, 2:, :] *= np.float32(2.0 ** -117)
        elif what == "filters":
            inputs["W"][:, 8:20] *= np.float32(2.0 ** -100)
        else:
            inputs["x"] *= np.float32(2.0 ** what[0])
            inputs["W"] *= np.float32(2.0 ** what[1])
        want = _oracle(orc, layer, inputs)
        for tm, waves in ((64, 4), (128, 8)):
            print("[case] tiles, scales", what, layer.name(), "nhwc" if nhwc else "nchw", tm, waves, flush=True)
            got = _run(layer, inputs, tm, waves, nhwc).astype(np.float64)
            for part in (np.abs(want) < 1e-25, np.abs(want) >= 1e-25):
                assert not part.any() or np.linalg.norm((got - want)[part] * 2.0 ** 60) <= 1.2e-6 * np.linalg.norm(want[part] * 2.0 ** 60)


# 1x1 layers whose pixels, all channels, stay in LDS: 512 pixel tiles, so that a workgroup takes two or more channel tiles.  P = 16368
# (tiles over two images) and 16384; 16383 allows NCHW no 16-byte stores and goes through the tile kernel there.  72 channels are
# the last in three parts, 73 and 76 the first in two, 288 the most that fit; 260 with few outputs go through the tile kernel.
@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("C,N", ((20, 136), (72, 136), (73, 136), (76, 136), (256, 136), (260, 136), (288, 264)))
@pytest.mark.parametrize("W", (124, 127, 128))
def test_1x1_layers_that_run_over_several_channel_tiles(nhwc, C, N, W):
    if nhwc and C % 4:
        pytest.skip("NHWC needs channel counts that are multiples of 4")
    layer = Layer(2, C, N, 32768 // 2 // W, W, 1, 1, 1, 1, 0)
    inputs = make_dense_inputs(layer, 84)
    rng = np.random.default_rng(7)
    bias = rng.standard_normal(layer.N, dtype=np.float32)
    residual = rng.standard_normal((layer.batch, layer.N, layer.Ho, layer.Wo), dtype=np.float32)
    plain = np.matmul(inputs["W"][:, :, 0, 0].astype(np.float64).T, inputs["x"].reshape(2, C, -1)).reshape(residual.shape)
    want = np.maximum(plain + bias[None, :, None, None] + residual, 0.0)
    for tm in (64, 128):
        for offset in (0,) if nhwc else (0, 1):
            print("[case] 1x1", layer.name(), "nhwc" if nhwc else "nchw", tm, offset, flush=True)
            assert_parity(_run(layer, inputs, tm, 4, nhwc, bias, residual, offset), want, "%s tile %d" % (layer.name(), tm))
        got = _run(layer, inputs, tm, 4, nhwc)
        # 9e-8 (72 terms, three parts) to 1.4e-7 (288, two): three times the larger; fp32 multiply-adds show 3.1e-7 at 288
        assert np.linalg.norm(got - plain) <= 4.2e-7 * np.linalg.norm(plain)


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer", (Layer(2, 160, 72, 13, 9, 1, 1, 1, 1, 0), Layer(2, 40, 72, 13, 9, 1, 1, 3, 1, 1)), ids=lambda l: l.name())
def test_values_far_from_those_that_set_the_scale(orc, layer, nhwc):
    """x is scaled by what a workgroup loads first.  Channels behind that up to 512 times larger fit in fp16 and larger ones do
    not; pixels down to 2^-19 of it keep all their bits and smaller ones do not.  Both sides of each line."""
    for what, e in [("channels", e) for e in (4, 6, 7, 9, 11, 40)] + [("pixels", -e) for e in (10, 17, 19, 21, 23, 25, 40)]:
        inputs = make_dense_inputs(layer, 85)
        if what == "channels":
            inputs["x"][:, -8:] *= np.float32(2.0 ** e)
        else:
            inputs["x"][0, :, 5:] *= np.float32(2.0 ** e)
        want = _oracle(orc, layer, inputs)
        for tm, waves in ((64, 4), (128, 8)):
            print("[case] tiles, far from the scale", what, e, layer.name(), "nhwc" if nhwc else "nchw", tm, waves, flush=True)
            err = _run(layer, inputs, tm, waves, nhwc) - want
            # pixel by pixel, each against its own size: 360 terms, as in test_tiles
            assert (np.linalg.norm(err, axis=1) <= 1.2e-6 * np.linalg.norm(want, axis=1)).all()


# 3x3: the tile kernel; 1x1: all channels in LDS, both layouts (P = 108), two and three parts
FP16_LAYERS = (Layer(2, 40, 72, 13, 9, 1, 1, 3, 1, 1), Layer(2, 160, 72, 12, 9, 1, 1, 1, 1, 0), Layer(130, 64, 136, 14, 16, 1, 1, 1, 1, 0))


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer", FP16_LAYERS, ids=lambda l: l.name())
@pytest.mark.parametrize("what", ("beyond_fp16", "late_channels", "wide_weights", "alone"))
def test_a_nan_explains_no_sums_but_its_own(orc, what, layer, nhwc):
    """One NaN beside finite values that fp16 does not hold at the scale the workgroup takes: values above 1023 where the NaN
    is among the first loads, channels 2^14 times larger behind the first loads, weights kept out of the parts."""
    inputs = make_dense_inputs(layer, 86)
    if what == "beyond_fp16":
        inputs["x"][0, :, 0, 3:6] *= np.float32(2.0 ** 12)
    elif what == "late_channels":
        inputs["x"][:, -8:] *= np.float32(2.0 ** 14)
    elif what == "wide_weights":
        inputs["W"][1:3, 7, layer.K // 2, layer.K // 2] = 2.0 ** 12, 2.0 ** -20
    inputs["x"][0, 3, 0, 0] = np.nan
    want = _oracle(orc, layer, inputs)
    for tm, waves in ((64, 4), (128, 8)):
        print("[case] tiles, one NaN,", what, layer.name(), "nhwc" if nhwc else "nchw", tm, waves, flush=True)
        got = _run(layer, inputs, tm, waves, nhwc)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        ok = ~np.isnan(want[0, 0])
        err, ref = (got - want)[0][:, ok], want[0][:, ok]
        assert (np.linalg.norm(err, axis=0) <= 1.2e-6 * np.linalg.norm(ref, axis=0)).all()
        assert (np.linalg.norm((got - want)[1:], axis=1) <= 1.2e-6 * np.linalg.norm(want[1:], axis=1)).all()


# What x or a weight may hold that no parts do, in 1x1 layers whose pixels stay in LDS
def _infinite_x(i):
    i["x"][0, 3, 4, 5] = np.inf


def _largest_x(i):
    i["x"][0, 3, 4, 5], i["x"][0, 9, 7, 2] = np.finfo(np.float32).max, -np.finfo(np.float32).max
    i["W"] = np.clip(i["W"], -0.5, 0.5)


def _nan_and_infinite_x(i):
    i["x"][0, 3, 4, 5], i["x"][0, 5, 1, 1] = np.inf, np.nan


def _largest_weight(i):
    i["W"][5, 7] = np.finfo(np.float32).max
    i["x"] *= np.float32(1e-12)


def _infinite_weight(i):
    i["W"][5, 7] = -np.inf


def _nan_weight(i):
    i["W"][5, 7] = np.nan


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer", FP16_LAYERS[1:], ids=lambda l: l.name())
@pytest.mark.parametrize("extreme", (_infinite_x, _largest_x, _nan_and_infinite_x, _largest_weight, _infinite_weight, _nan_weight), ids=lambda f: f.__name__[1:])
def test_1x1_layers_in_lds_with_values_that_no_parts_hold(orc, extreme, layer, nhwc):
    inputs = make_dense_inputs(layer, 89)
    extreme(inputs)
    with np.errstate(invalid="ignore"):
        want = _oracle(orc, layer, inputs)
    for tm in (64, 128):                                 # one and two channel blocks to a wavefront where there are two parts
        print("[case] 1x1 in LDS,", extreme.__name__, layer.name(), "nhwc" if nhwc else "nchw", tm, flush=True)
        got = _run(layer, inputs, tm, 4, nhwc, in_lds=True, parts="fp16x3" if layer.C <= 72 else "fp16x2")
        finite = np.isfinite(want)
        assert (extreme in (_largest_x, _largest_weight)) == finite.all()
        assert np.array_equal(got[~finite], want[~finite].astype(np.float32), equal_nan=True)
        reached = finite & (np.abs(want) > 1e25 if extreme is not _largest_weight else np.abs(want) > 1e10)
        for part in (reached, finite & ~reached):        # sums of at most 160 terms, as in test_tiles
            assert np.linalg.norm(got[part] - want[part]) <= 1.2e-6 * np.linalg.norm(want[part])


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer", FP16_LAYERS, ids=lambda l: l.name())
def test_channels_that_the_weights_bring_to_one_size(orc, layer, nhwc):
    """x in channels of very different size, which the weights undo: the result is that of the same layer without.  Parts of
    fp16 keep x and the weights to an absolute accuracy only, which shows from some 2^20 between the channels on."""
    for bits in (8, 16, 20, 24, 28, 34, 40, 60):
        inputs = make_dense_inputs(layer, 87)
        for of in ("even", "late"):
            s = np.ones(layer.C, np.float32)
            s[slice(None, None, 2) if of == "even" else slice(None, layer.C // 2)] = 2.0 ** bits
            there = dict(x=inputs["x"] * s[None, :, None, None], W=inputs["W"] / s[:, None, None, None])
            if of == "even":
                there["x"][0, ::2, :, 4:] = 0            # pixels of nothing but the smaller channels
            want = _oracle(orc, layer, there)
            for tm, waves in ((64, 4), (128, 8)):
                print("[case] tiles, channels 2^%d apart" % bits, of, layer.name(), "nhwc" if nhwc else "nchw", tm, waves, flush=True)
                err = _run(layer, there, tm, waves, nhwc) - want
                assert (np.linalg.norm(err, axis=1) <= 1.2e-6 * np.linalg.norm(want, axis=1)).all()


def _small_quarter(i):               # what one of the four wavefronts that share NCHW pixels brings
    for c in range(4, i["x"].shape[1], 16):
        i["x"][:, c:c + 4] *= np.float32(2.0 ** -30)


def _larger_late(i):                 # behind what sets the scale
    i["x"][:, -8:] *= np.float32(200.0)


def _dead(i):                        # filters without a weight, images without a value
    i["W"][:, ::2] = 0
    i["W"][:, :17] = 0
    i["x"][1::2] = 0


ORDINARY = (_small_quarter, _larger_late, _dead)


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer", (Layer(8, 128, 128, 28, 28, 1, 1, 3, 1, 1), Layer(8, 128, 512, 28, 28, 1, 1, 1, 1, 0)), ids=lambda l: l.name())
@pytest.mark.parametrize("values", ORDINARY, ids=lambda f: f.__name__[1:])
def test_finite_inputs_that_fp16_holds_cost_the_usual_time(values, layer, nhwc):
    """They are not computed again in fp32, which takes several times as long."""
    import torch
    from paper_2211_03715_amd.layer import DenseConv2d
    dev = torch.device("cuda:0")
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a.transpose(0, 2, 3, 1) if nhwc else a)).to(dev)
    usual = make_dense_inputs(layer, 88)
    other = {k: v.copy() for k, v in usual.items()}
    values(other)
    conv = DenseConv2d(layer, 0, B.make_tuning(tile_h=64, tile_w=64, waves=(4,) * 3), B.LAYOUT_NHWC if nhwc else B.LAYOUT_NCHW)
    try:
        us = []
        y = torch.empty(conv.out_shape(), device=dev)
        for inputs in (usual, other):
            W = torch.from_numpy(inputs["W"]).to(dev)
            conv.pack(W)
            launch = conv.bind(put(inputs["x"]), y)
            gpu_us(launch)
            us.append(gpu_us(launch))
        print("[case] tiles,", values.__name__, layer.name(), "nhwc" if nhwc else "nchw", "%.1f us, usually %.1f" % (us[1], us[0]), flush=True)
        assert us[1] <= 1.5 * us[0]
        if values is _dead:
            y = y.permute(0, 3, 1, 2) if nhwc else y
            assert not y[:, ::2].any() and not y[:, :17].any() and not y[1::2].any() and y[0, 17].any()
    finally:
        conv.close()


@pytest.mark.parametrize("nhwc", (False, True), ids=("nchw", "nhwc"))
@pytest.mark.parametrize("layer,pixel", ((Layer(1, 128, 64, 10, 10, 1, 1, 3, 1, 1), 97), (Layer(1, 256, 136, 2, 36, 1, 1, 1, 1, 0), 70),
                                         (Layer(1, 64, 64, 1, 1, 1, 1, 3, 1, 1), None)), ids=lambda v: v.name() if isinstance(v, Layer) else "")
def test_one_sum_that_is_small_by_chance_has_no_tile_computed_again(orc, layer, pixel, nhwc):
    """A channel that one of the last pixels, alone in its lane, happens to give nothing.  The other channels would not keep their bits if
    the tile were computed again.  A single pixel in all is judged by itself: only its values are checked."""
    inputs = make_dense_inputs(layer, 90)
    p = pixel or 0
    x = np.pad(inputs["x"][0].astype(np.float64), ((0, 0), (layer.pad,) * 2, (layer.pad,) * 2))
    h, w = p // layer.W, p % layer.W
    v = x[:, h:h + layer.K, w:w + layer.K].ravel()
    there = dict(inputs, W=inputs["W"].copy())
    u = inputs["W"][:, 7].astype(np.float64).ravel()
    there["W"][:, 7] = (u - v * (v @ u) / (v @ v)).reshape(there["W"][:, 7].shape)
    others = np.arange(layer.N) != 7
    for tm, waves in ((64, 4), (64, 8), (128, 4)):
        print("[case] tiles, small by chance", layer.name(), "nhwc" if nhwc else "nchw", tm, waves, flush=True)
        got, clean = _run(layer, there, tm, waves, nhwc), _run(layer, inputs, tm, waves, nhwc)
        assert abs(got[0, 7, h, w]) < 1e-5
        assert pixel is None or np.array_equal(got[:, others], clean[:, others])
        assert_parity(got, _oracle(orc, layer, there), layer.name())
