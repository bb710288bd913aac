"""The untuned launches on layouts whose lane-blocks hold less than a line per
entry (host computation): loads stay cached, below 64 bytes stores too, and the
layouts of whole lines keep theirs."""
import pytest

import paper_1710_09409_amd as su3

F64, F32, F16, C12 = su3.SU3_F64, su3.SU3_F32, su3.SU3_F16_F32ACC, su3.SU3_C12_F32
VN, AOSOA, SOA = su3.SU3_LAYOUT_VNODE, su3.SU3_LAYOUT_AOSOA, su3.SU3_LAYOUT_SOA
MUL, SHIFT, COPY = su3.SU3_EXPR_MUL, su3.SU3_EXPR_MUL_SHIFTED, su3.SU3_EXPR_CSHIFT
BIG = (48, 48, 48, 48)


def _nt(expr, prec, layout, lanes, dims=BIG):
    su3.su3_launch_reset()
    return su3.su3_launch_get(expr, prec, layout, lanes, dims).nontemporal


@pytest.mark.parametrize("prec,layout,lanes", [
    (F64, VN, 2), (F32, VN, 2), (F16, VN, 2), (C12, VN, 2), (F32, VN, 4), (F16, VN, 4),
    (C12, VN, 4), (F16, VN, 8), (F16, AOSOA, 8)])
def test_pieces_of_less_than_64_bytes(prec, layout, lanes):
    assert _nt(MUL, prec, layout, lanes) == 0
    assert _nt(su3.SU3_EXPR_BATCH + MUL, prec, layout, lanes) == 0
    for expr in (SHIFT, COPY):
        assert _nt(expr, prec, layout, lanes) & 1 == 0


@pytest.mark.parametrize("prec,layout,lanes", [(F64, VN, 4), (F32, VN, 8), (F32, AOSOA, 8),
                                               (C12, AOSOA, 8), (F16, AOSOA, 16)])
def test_pieces_of_64_bytes(prec, layout, lanes):
    assert _nt(MUL, prec, layout, lanes) == 2
    assert _nt(su3.SU3_EXPR_BATCH + MUL, prec, layout, lanes) == 0
    for expr in (SHIFT, COPY):
        assert prec != F64 or _nt(expr, prec, layout, lanes) & 1 == 0


@pytest.mark.parametrize("layout,lanes", [(SOA, 0), (AOSOA, 64), (VN, 16)])
def test_whole_lines(layout, lanes):
    for expr in (MUL, SHIFT, COPY, su3.SU3_EXPR_BATCH + MUL):
        assert _nt(expr, F64, layout, lanes) & 1 == 1


def test_double_product_streams_its_stores_late():
    """From 512 MB on: below, nontemporal stores are as fast or faster."""
    assert _nt(SHIFT, F64, SOA, 0, (28, 28, 28, 28)) == 3
    assert _nt(SHIFT, F64, SOA, 0, (32, 32, 32, 32)) == 3
    assert _nt(SHIFT, F64, SOA, 0, (36, 36, 36, 36)) == 7
