"""The untuned launch of the hopping term by lattice, precision and layout
(host computation): one wave per hop where the walks suffer from the extents,
two-buffer tiles where a line holds more of other entries than of its own,
ranges per XCD only where no CU gets a workgroup more."""
import pytest

import paper_1710_09409_amd as su3

F64, F32, C12 = su3.SU3_F64, su3.SU3_F32, su3.SU3_C12_F32
SOA, AOS, AOSOA, VN = (su3.SU3_LAYOUT_SOA, su3.SU3_LAYOUT_AOS, su3.SU3_LAYOUT_AOSOA,
                       su3.SU3_LAYOUT_VNODE)


def _plan(prec, layout, lanes, dims):
    su3.su3_launch_reset()
    return su3.su3_launch_get(su3.SU3_EXPR_DSLASH, prec, layout, lanes, dims)


@pytest.mark.parametrize("prec,layout,lanes,dims,hops", [
    (C12, VN, 16, (28, 28, 28, 28), True), (F32, VN, 16, (28, 28, 28, 28), True),
    (C12, VN, 8, (28, 28, 28, 28), True), (F32, SOA, 0, (26, 26, 26, 26), True),
    (C12, SOA, 0, (28, 28, 28, 28), True), (F32, AOSOA, 64, (22, 22, 22, 44), True),
    (C12, VN, 16, (32, 32, 32, 18), False), (F32, VN, 2, (28, 28, 28, 28), False),
    (F32, SOA, 0, (32, 32, 32, 32), False), (F64, SOA, 0, (26, 26, 26, 26), False),
])
def test_one_wave_per_hop(prec, layout, lanes, dims, hops):
    c = _plan(prec, layout, lanes, dims)
    assert ((c.schedule, c.tile_sites, c.sites_per_lane) == (0, 1, 8)) == hops


@pytest.mark.parametrize("dims", [(24, 24, 24, 24), (28, 28, 28, 28), (32, 32, 32, 32),
                                  (40, 40, 40, 40), (48, 48, 48, 48)])
def test_short_runs(dims):
    two_buffers = dims[0] * 9 * 12 * 16 * 2 <= 160 * 1024
    assert _plan(F64, AOS, 0, dims).schedule in ((18, 28) if two_buffers else (17, 27))
    for prec in (F64, F32):
        c = _plan(prec, VN, 2, dims)
        assert c.xcd_remap == 0
        assert prec == F64 or c.schedule in (16, 18)


def test_walks():
    for layout, lanes in ((SOA, 0), (AOSOA, 8), (AOSOA, 64)):
        c = _plan(F32, layout, lanes, (28, 28, 28, 28))
        assert (c.schedule, c.tile_sites) == (16, 6)
        # 100 tiles in 5 walks: 65 of the 500 workgroups for each XCD's 32 CUs
        assert _plan(F32, layout, lanes, (20, 40, 40, 40)).xcd_remap == 0
    # outer rows of 17 sites in pieces of one
    c = _plan(F32, VN, 16, (34, 34, 34, 34))
    assert (c.schedule, c.tile_sites, c.xcd_remap) == (16, 7, 0)
