"""What the selector may and may not choose, on the CPU."""
import numpy as np
import pytest

from paper_2211_03715_amd import autotune as A
from paper_2211_03715_amd import binding as B
from paper_2211_03715_amd.workloads import Layer


@pytest.fixture(scope="module", autouse=True)
def lib():
    B.load()


def _auto(layout=B.LAYOUT_NCHW, tuning=None, **kw):
    dims = dict(batch=256, C=128, N=128, H=28, W=28, R1=32, R2=32, K=3, stride=1, pad=1)
    dims.update(kw)
    return B.tdc_select_tuning(B.make_shape(layout=layout, **dims), tuning=tuning)


def _is_bf16(t):
    return t.variant == B.VARIANT_CHAIN and t.mb[1] == 3


@pytest.mark.parametrize("layout", (B.LAYOUT_NCHW, B.LAYOUT_NHWC), ids=("nchw", "nhwc"))
def test_sums_of_one_or_two_terms_stay_in_fp32(layout):
    """The split products are less exact than fp32 multiply-adds there."""
    assert _is_bf16(_auto(layout)) and _is_bf16(_auto(layout, C=4, R1=20, R2=3))
    few = [dict(R2=2), dict(R1=2, K=1, pad=0)] + ([dict(C=2)] if layout == B.LAYOUT_NCHW else [])
    for kw in few:
        assert not _is_bf16(_auto(layout, **kw)), kw
    dense = lambda **kw: _auto(layout, B.make_tuning(variant=B.VARIANT_DENSE), **kw).tile_h
    assert dense()
    if layout == B.LAYOUT_NCHW:
        assert not dense(C=1, K=1, pad=0) and not dense(C=2, K=1, pad=0)


def test_auto_honours_the_fields_a_caller_sets():
    """Zero in a field means the selector's choice, and only zero does: each field set alone comes back, or the tuning is
    refused.  (wavefronts and register tiles of stage 1 and of the pixels; the other stages' are not every kernel's)"""
    layers = (dict(), dict(batch=32, C=256, N=256, H=14, W=14, R1=64, R2=64), dict(batch=3, C=100, N=152, H=37, W=29, R1=24, R2=40, K=5, pad=2),
              dict(batch=1, C=64, N=64, H=224, W=224, R1=64, R2=32))
    for kw in layers:
        for layout in (B.LAYOUT_NCHW, B.LAYOUT_NHWC):
            for field, values in (("tile_h", (2, 7, 8)), ("tile_w", (4, 8, 14)), ("waves", (2, 4, 8)), ("mb", (1, 2)), ("pb", (1, 2))):
                for v in values:
                    forced = B.make_tuning(**{field: v if field.startswith("tile") else (v, 0, 0)})
                    try:
                        t = _auto(layout, forced, **kw)
                    except B.TdcError as e:
                        assert e.status == B.TDC_ERR_BAD_TUNING
                        continue
                    if field.startswith("tile") and t.variant in (B.VARIANT_SPLIT, B.VARIANT_MERGED):
                        continue                                # these have no spatial tile
                    got = getattr(t, field)
                    assert (got if field.startswith("tile") else got[0]) == v, (kw, layout, field, v, t.as_dict())
            assert _auto(layout, B.make_tuning(tile_h=4, tile_w=4, pb=(1, 0, 0)), **kw).pb[0] == 1


@pytest.mark.parametrize("fields", (dict(tile_h=8), dict(tile_h=96), dict(tile_h=64), dict(tile_w=64), dict(tile_h=14, tile_w=14),
                                    dict(tile_h=64, tile_w=64, mb=(0, 2, 0)), dict(tile_h=128, tile_w=64, pb=(0, 4, 0))), ids=str)
def test_a_dense_tuning_without_a_whole_tile_means_the_latency_kernel(fields):
    """tile_h and tile_w are fields the latency kernel has never had: alone, small, or beside its register tile they say nothing."""
    shape = B.make_shape(batch=2, C=64, N=128, H=28, W=28, R1=1, R2=1, K=3, stride=1, pad=1)
    plain = {k: v for k, v in fields.items() if not k.startswith("tile")}
    want = B.tdc_select_tuning(shape, tuning=B.make_tuning(variant=B.VARIANT_DENSE, **plain)).as_dict()
    assert B.tdc_select_tuning(shape, tuning=B.make_tuning(variant=B.VARIANT_DENSE, **fields)).as_dict() == want
    for k, v in plain.items():
        assert want[k][1] == v[1] and want["tile_h"] == 0
    full = dict(mb=(2, 2, 2), pb=(1, 1, 1), waves=(4, 4, 4), **{k: v for k, v in fields.items() if k.startswith("tile")})
    assert B.tdc_model_terms(shape, B.make_tuning(variant=B.VARIANT_DENSE, **full))[0] == "dense"


def test_every_choice_has_an_estimate_that_a_caller_can_rebuild():
    """Terms and table of whatever the selector picks, the bf16 kernels included, have the same length, and the product is the
    estimate: of two tunings of one kernel the pick's is the lower one."""
    tables = A.read_coefficients()
    for layout in (B.LAYOUT_NCHW, B.LAYOUT_NHWC):
        shape = B.make_shape(256, 128, 128, 28, 28, 32, 32, 3, 1, 1, layout)
        pick = B.tdc_select_tuning(shape)
        assert _is_bf16(pick)
        model, names, terms = B.tdc_model_terms(shape, pick)
        assert len(tables[model]) == len(names) == len(terms) and sum(1 for t in terms if t) == 4
        est = float(np.dot(tables[model], terms))
        d = pick.as_dict()
        for th, tw, mb1 in ((2, 28, 2), (4, 28, 1), (4, 16, 2), (8, 14, 2)):
            other = B.make_tuning(variant=B.VARIANT_CHAIN, tile_h=th, tile_w=tw, waves=(4,) * 3, mb=(mb1, 3, 1), pb=tuple(d["pb"]))
            assert est <= float(np.dot(tables[model], B.tdc_model_terms(shape, other)[2])) + 1e-9
        dense = B.make_tuning(variant=B.VARIANT_DENSE)
        pick = B.tdc_select_tuning(shape, tuning=dense)
        model, names, terms = B.tdc_model_terms(shape, pick)
        assert model == "dense_tile" and len(tables[model]) == len(names) == len(terms)
        est = float(np.dot(tables[model], terms))
        for tm, waves in ((64, 4), (64, 8), (128, 4), (128, 8)):
            other = B.make_tuning(variant=B.VARIANT_DENSE, tile_h=tm, tile_w=64, waves=(waves,) * 3, mb=(1,) * 3, pb=(1,) * 3)
            assert est <= float(np.dot(tables[model], B.tdc_model_terms(shape, other)[2])) + 1e-9


def test_the_exhaustive_search_lists_the_kernels_the_selector_takes():
    """The searched optimum can only be no worse than AUTO if AUTO's kernels are among the candidates."""
    for L in (Layer(32, 128, 128, 28, 28, 32, 32, 3, 1, 1), Layer(32, 256, 256, 14, 14, 64, 64, 3, 1, 1), Layer(1, 64, 64, 224, 224, 64, 32, 3, 1, 1),
              Layer(8, 128, 256, 56, 56, 32, 64, 3, 2, 1)):
        pick = _auto(**L.asdict())
        assert _is_bf16(pick)
        listed = {(c["variant"], c.get("tile_h"), c.get("tile_w"), c["mb"][0], c["mb"][1], c.get("pb", (0,))[0]) for c in A.candidates(L)}
        assert (pick.variant, pick.tile_h, pick.tile_w, pick.mb[0], pick.mb[1], pick.pb[0]) in listed, pick.as_dict()
    assert not any(c["variant"] == B.VARIANT_CHAIN and c["mb"][1] == 3 for c in A.candidates(Layer(32, 512, 512, 7, 7, 128, 128, 3, 1, 1)))


def test_where_few_pixels_leave_layers_with_the_fp32_kernels():
    """Below 16 output pixels per compute unit: not 1x1 layers at stride 1, nor narrow NCHW ones whose rows are no multiple of 4;
    the others are.  (26x38, 112 -> 160: 11.0 us on the bf16 matrix cores, 9.5 in fp32)"""
    few = dict(batch=3, C=112, N=160, H=26, W=38, R1=20, R2=32)
    assert not _is_bf16(_auto(**few))
    assert _is_bf16(_auto(batch=6, C=137, N=100, H=29, W=18, R1=54, R2=41))                 # four blocks of R1
    assert _is_bf16(_auto(batch=10, C=204, N=219, H=20, W=20, R1=60, R2=76))                # rows of quads
    assert _is_bf16(_auto(B.LAYOUT_NHWC, batch=2, C=124, N=136, H=43, W=45, R1=22, R2=33))
    one = dict(batch=28, C=372, N=284, H=12, W=11, R1=49, R2=50, K=1, pad=0)
    assert not _is_bf16(_auto(**one)) and not _is_bf16(_auto(B.LAYOUT_NHWC, **one))


def test_tiles_of_large_nchw_images_without_16_byte_rows():
    """179x179: whole pixel blocks in a tile's rows (51.6 us) instead of 9 pixels (62.6)."""
    t = _auto(batch=2, C=96, N=144, H=179, W=179, R1=17, R2=34)
    assert _is_bf16(t) and t.tile_w % 16 == 0 and t.tile_h * t.tile_w <= 128


def test_short_dense_contractions_with_4_byte_stores_stay_with_the_latency_kernel():
    dense = lambda **kw: _auto(tuning=B.make_tuning(variant=B.VARIANT_DENSE), **dict(dict(K=1, pad=0, R1=1, R2=1), **kw)).tile_h
    assert not dense(batch=2, C=32, N=80, H=214, W=214, stride=2) and not dense(batch=5, C=26, N=104, H=63, W=63)
    assert dense(batch=5, C=26, N=104, H=64, W=64) and dense(batch=5, C=160, N=104, H=63, W=63)


def test_dense_tiles_take_weights_up_to_2_GiB_in_three_parts():
    """What a kernel addresses behind one descriptor is its weights in parts, six bytes each at most: up to 357 million of them.  The copy in
    fp32 beside them has a descriptor of its own."""
    for C, N, K, fits in ((5120, 5120, 3, True), (16384, 16384, 1, True), (20480, 18432, 1, False), (6400, 6400, 3, False)):
        shape = B.make_shape(1, C, N, 64, 64, 1, 1, K, 1, K // 2)
        assert (C * N * K * K * 6 < 2 ** 31) == fits
        forced = B.make_tuning(variant=B.VARIANT_DENSE, tile_h=64, tile_w=64, waves=(4, 4, 4))
        if fits:
            assert B.tdc_select_tuning(shape, tuning=forced).tile_h == 64
            assert B.tdc_select_tuning(shape, tuning=B.make_tuning(variant=B.VARIANT_DENSE)).tile_h >= 64
        else:
            with pytest.raises(B.TdcError):
                B.tdc_select_tuning(shape, tuning=forced)
            assert B.tdc_select_tuning(shape, tuning=B.make_tuning(variant=B.VARIANT_DENSE)).tile_h == 0
