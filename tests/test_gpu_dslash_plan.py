"""Walks whose workgroups are dealt to the XCDs in ranges of tiles, chosen by
the lattice's extents: ragged tiles, a number of tiles that eight does and does
not divide, short last walks, virtual nodes.  Bit for bit one site per lane."""
import pytest
import torch

import paper_1710_09409_amd as su3
from test_gpu_dslash_hops import AOSOA, C12, F32, F64, ONE_SITE, SOA, VN, _fields, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lp,dims,layout,lanes,simd,remap", [
    (F64, (32, 32, 32, 12), SOA, 0, None, 2),
    (F64, (30, 34, 26, 14), SOA, 0, None, None),     # ragged in y, z and t
    (F32, (64, 24, 20, 13), AOSOA, 64, None, None),
    (C12, (36, 36, 36, 9), AOSOA, 16, None, None),   # 81 tiles
    (F32, (28, 30, 28, 16), SOA, 0, None, None),
    (C12, (32, 32, 32, 18), VN, 16, (2, 2, 2, 2), None),
    (F64, (24, 28, 26, 22), VN, 8, (2, 2, 2, 1), None),
])
def test_planned_ranges(lp, dims, layout, lanes, simd, remap):
    f = _fields(dims, lp, layout, lanes, simd)
    want = _run(f, dims, lp, layout, lanes, ONE_SITE)
    su3.su3_launch_reset()
    plan = su3.su3_launch_get(su3.SU3_EXPR_DSLASH, lp, layout, lanes, dims).as_dict()
    assert remap is None or plan["xcd_remap"] == remap
    assert torch.equal(_run(f, dims, lp, layout, lanes, None), want)
    for x in (0, 1, 2):
        cfg = dict(plan, xcd_remap=x)
        assert torch.equal(_run(f, dims, lp, layout, lanes, cfg), want), x
