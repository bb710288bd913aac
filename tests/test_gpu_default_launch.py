"""The launch an untuned call takes changes with its bytes, precision, layout
and plane spacing.  On both sides of every line the result is bit for bit
that of a plain launch (64 lanes per workgroup, cached, uncapped), padding
included."""
import pytest
import torch

import paper_1710_09409_amd as su3

pytestmark = pytest.mark.gpu

SOA, AOSOA, AOS = su3.SU3_LAYOUT_SOA, su3.SU3_LAYOUT_AOSOA, su3.SU3_LAYOUT_AOS
F64, F32, F16, C12 = su3.SU3_F64, su3.SU3_F32, su3.SU3_F16_F32ACC, su3.SU3_C12_F32
DTYPE = {F64: torch.float64, F32: torch.float32, F16: torch.float16, C12: torch.float32}
MUL, MUL3, MULADD = su3.SU3_EXPR_MUL, su3.SU3_EXPR_MUL3, su3.SU3_EXPR_MULADD
PLAIN = dict(block=64, persistent=0, nontemporal=0, xcd_remap=0, lds_stage=0, tile_sites=4096,
             occupancy=0, schedule=1, sites_per_lane=0)


def _fields(n, dims, prec, layout, lanes):
    out = []
    for k in range(n):
        f = su3.field_tensor(dims, prec, layout, lanes)
        g = torch.Generator(device="cuda")
        g.manual_seed(17 + k)
        t = f.owner.view(DTYPE[prec])
        t.copy_(torch.randn(t.shape, generator=g, device="cuda").to(t.dtype))
        out.append(f)
    return out


def _same(key, prec, layout, lanes, dims, n_ops, call):
    *ops, z = _fields(n_ops + 1, dims, prec, layout, lanes)
    before = z.owner.clone()
    su3.su3_launch_reset()
    call(z, ops)
    got = z.owner.clone()
    z.owner.copy_(before)
    su3.su3_launch_set(key, prec, layout, lanes, dims, dict(PLAIN, schedule=int(layout != AOS)))
    try:
        call(z, ops)
    finally:
        su3.su3_launch_reset()
    assert not torch.equal(got, before)
    assert torch.equal(got, z.owner)


@pytest.mark.parametrize("expr,prec,layout,lanes,dims", [
    (MUL, F64, SOA, 0, (7, 9, 11, 13)),        # small, ragged
    (MUL, F64, SOA, 0, (24, 24, 24, 26)),      # 155 MB: cached
    (MUL, F64, SOA, 0, (24, 24, 24, 27)),      # 161 MB: streaming
    (MUL, F64, SOA, 0, (16, 16, 16, 32)),      # planes 2 MiB apart
    (MUL, F32, SOA, 0, (32, 32, 32, 32)),      # planes 8 MiB apart, streaming
    (MUL, F32, AOSOA, 64, (48, 48, 48, 23)),   # over half a GB
    (MUL3, F16, SOA, 0, (21, 19, 23, 25)),     # half, ragged, cached
    (MULADD, F16, AOSOA, 16, (32, 32, 32, 31)),  # half, four operands, streaming
    (MUL, C12, SOA, 0, (33, 31, 35, 36)),      # two-row, streaming
    (MUL, F32, AOS, 0, (24, 24, 24, 25)),
    (MULADD, F64, AOS, 0, (16, 16, 17, 19)),
    (MULADD, F32, AOS, 0, (24, 24, 24, 35)),   # AoS, streaming
    (MUL, F64, AOS, 0, (24, 24, 24, 27)),
])
def test_site_local(expr, prec, layout, lanes, dims):
    _same(expr, prec, layout, lanes, dims, su3.N_OPERANDS[expr],
          lambda z, ops: su3.su3_fused_eval(z, expr, ops, torch.cuda.current_stream()))


@pytest.mark.parametrize("prec,layout,lanes,dims", [
    (F64, SOA, 0, (5, 7, 9, 11)), (F64, SOA, 0, (24, 24, 24, 17)), (F64, AOSOA, 64, (24, 24, 24, 35)),
    (F64, SOA, 0, (32, 32, 32, 37)), (F32, SOA, 0, (24, 24, 24, 48)), (F16, SOA, 0, (24, 24, 24, 24)),
    (C12, AOSOA, 8, (32, 32, 32, 32)), (F64, AOS, 0, (9, 9, 9, 9)), (F16, AOS, 0, (9, 9, 9, 9)),
])
def test_shifted(prec, layout, lanes, dims):
    s = torch.cuda.current_stream()
    _same(su3.SU3_EXPR_CSHIFT, prec, layout, lanes, dims, 1,
          lambda z, ops: su3.su3_cshift(z, ops[0], 0, 1, s))
    _same(su3.SU3_EXPR_MUL_SHIFTED, prec, layout, lanes, dims, 2,
          lambda z, ops: su3.su3_mult_shifted(z, ops[0], ops[1], 3, -1, s))


@pytest.mark.parametrize("count", [1, 3, 40])
def test_batch(count):
    """Tiles of 128 sites, launched directly, replayed, and captured by the
    caller into a graph."""
    s = torch.cuda.current_stream()
    shapes = [((2, 3, 5, 7), F64), ((8, 8, 8, 8), C12), ((12, 12, 12, 13), F64)]
    zs, ops, want = [], [], []
    for i in range(count):
        dims, prec = shapes[i % 3]
        x, y, z = _fields(3, dims, prec, SOA, 0)
        su3.su3_mult(z, x, y, s)
        want.append(z.owner.clone())
        zs.append(z)
        ops.append([x, y])
    b = su3.su3_batch_create([MUL] * count, zs, ops, s)
    side = torch.cuda.Stream()
    side.wait_stream(s)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        su3.su3_batch_launch(b, side)
    for replay in (lambda: su3.su3_batch_launch(b, s), graph.replay, graph.replay,
                   lambda: su3.su3_batch_launch(b, s)):
        for z in zs:
            z.owner[: z.owner.numel() // 2].zero_()
        replay()
        torch.cuda.synchronize()
        for z, w in zip(zs, want):
            n = su3.volume(z.dims) * 2 * (8 if z.prec == F64 else 4)  # entry 0, no padding
            assert torch.equal(z.owner[:n], w[:n])
