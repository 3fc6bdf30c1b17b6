"""What the selector may and may not choose, on the CPU."""
import pytest

from paper_2211_03715_amd import binding as B


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
