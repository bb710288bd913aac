"""The hopping term with one wave per hop, and the launch that the lattice's
extents choose: bit for bit the one-site-per-lane kernel, and the oracle's
values within the single- and double-precision bounds of the other kernels."""
import pytest
import torch

import oracle
import testgen
import paper_1710_09409_amd as su3
from test_gpu_dslash import assert_dslash, magnitude

pytestmark = pytest.mark.gpu

SOA, AOSOA, AOS = su3.SU3_LAYOUT_SOA, su3.SU3_LAYOUT_AOSOA, su3.SU3_LAYOUT_AOS
VN = su3.SU3_LAYOUT_VNODE
F64, F32, C12 = su3.SU3_F64, su3.SU3_F32, su3.SU3_C12_F32
ONE_SITE = dict(block=64, persistent=0, nontemporal=0, xcd_remap=0, lds_stage=0, tile_sites=1,
                occupancy=0, schedule=0, sites_per_lane=0)
HOPS = dict(ONE_SITE, sites_per_lane=8)


def _fields(dims, lp, layout, lanes, simd):
    sp = F64 if lp == F64 else F32
    out = []
    for k in range(6):
        prec, kind = (sp, su3.SU3_KIND_SPINOR) if k < 2 else (lp, su3.SU3_KIND_MATRIX)
        if layout == VN:
            f = su3.vnode_tensor(dims, prec, simd, kind)
        elif k < 2:
            f = su3.spinor_tensor(dims, prec, layout, lanes)
        else:
            f = su3.field_tensor(dims, prec, layout, lanes)
        if k:
            g = torch.Generator(device="cuda")
            g.manual_seed(29 + k)
            t = f.owner.view(torch.float64 if prec == F64 else torch.float32)
            t.copy_(torch.randn(t.shape, generator=g, device="cuda", dtype=t.dtype))
        out.append(f)
    return out


def _run(fields, dims, lp, layout, lanes, cfg):
    out, inp, *links = fields
    out.owner.fill_(0x5a)
    su3.su3_launch_reset()
    if cfg:
        su3.su3_launch_set(su3.SU3_EXPR_DSLASH, lp, layout, lanes, dims, cfg)
    try:
        su3.su3_dslash(out, links, inp, torch.cuda.current_stream())
    finally:
        su3.su3_launch_reset()
    return out.owner.clone()


@pytest.mark.parametrize("lp", [F64, F32, C12])
@pytest.mark.parametrize("dims,layout,lanes,simd", [
    ((1, 1, 1, 1), SOA, 0, None), ((3, 3, 7, 1), SOA, 0, None),  # 63 sites
    ((4, 4, 2, 2), AOSOA, 8, None), ((5, 13, 1, 1), SOA, 0, None),  # 64, 65
    ((3, 5, 7, 11), AOSOA, 16, None), ((3, 5, 7, 11), AOS, 0, None),
    ((6, 4, 6, 10), VN, 4, (1, 1, 2, 2)), ((4, 4, 8, 6), VN, 16, (2, 2, 2, 2)),
    ((2, 3, 5, 7), VN, 1, (1, 1, 1, 1)), ((16, 16, 16, 9), SOA, 0, None),
])
def test_hops_equal_one_site(lp, dims, layout, lanes, simd):
    f = _fields(dims, lp, layout, lanes, simd)
    want = _run(f, dims, lp, layout, lanes, ONE_SITE)
    for x in (0, 1):
        for nt in (0, 1, 2, 3):
            cfg = dict(HOPS, xcd_remap=x, nontemporal=nt)
            assert torch.equal(_run(f, dims, lp, layout, lanes, cfg), want), (x, nt)
    assert torch.equal(_run(f, dims, lp, layout, lanes, None), want)


@pytest.mark.parametrize("lp,dims,layout,lanes,simd", [
    (F64, (24, 24, 25, 25), SOA, 0, None), (F64, (24, 24, 25, 26), SOA, 0, None),  # the line
    (F64, (33, 31, 20, 19), AOSOA, 64, None), (F32, (40, 25, 21, 22), SOA, 0, None),
    (C12, (25, 25, 20, 33), AOSOA, 32, None), (F64, (130, 12, 14, 20), SOA, 0, None),
    (F32, (24, 20, 24, 16), VN, 4, (1, 1, 2, 2)), (F64, (28, 24, 24, 26), VN, 16, (2, 2, 2, 2)),
    (F64, (40, 20, 20, 14), AOS, 0, None), (F32, (9, 9, 9, 600), SOA, 0, None),
])
def test_planned_launch_equals_one_site(lp, dims, layout, lanes, simd):
    f = _fields(dims, lp, layout, lanes, simd)
    want = _run(f, dims, lp, layout, lanes, ONE_SITE)
    assert torch.equal(_run(f, dims, lp, layout, lanes, None), want)


@pytest.mark.parametrize("lp", [F64, F32])
def test_hops_against_oracle(lp):
    dims, s = (4, 6, 3, 5), torch.cuda.current_stream()
    V = testgen.volume(dims)
    hu = [testgen.su3_field(V, field_id=testgen.FID_U0 + mu) for mu in range(4)]
    hin = testgen.spinor_field(V)
    links = []
    for h in hu:
        u = su3.field_tensor(dims, lp, SOA)
        su3.su3_field_upload(u, h, s)
        links.append(u)
    inp, out = su3.spinor_tensor(dims, lp, SOA), su3.spinor_tensor(dims, lp, SOA)
    su3.su3_field_upload(inp, hin, s)
    su3.su3_launch_reset()
    assert su3.su3_launch_get(su3.SU3_EXPR_DSLASH, lp, SOA, 0, dims).sites_per_lane == 8
    su3.su3_dslash(out, links, inp, s)
    got = su3.su3_field_download(out, s)
    qu = [su3.su3_field_download(u, s) for u in links]
    psi = su3.su3_field_download(inp, s)
    want = oracle.get().dslash(qu, psi, dims)
    assert_dslash(lp, lp, got, want, magnitude(qu, psi, dims), "one wave per hop")
