"""Untuned batches: an item whose entry planes are 2 to 16 MiB apart has its
tiles dealt to the XCDs in ranges, and block, tile and schedule follow the
precision of most bytes.  Bit for bit the single calls, for items whose tile
counts eight does and does not divide, first and last in the table."""
import pytest
import torch

import paper_1710_09409_amd as su3

pytestmark = pytest.mark.gpu

F64, F32, F16, C12 = su3.SU3_F64, su3.SU3_F32, su3.SU3_F16_F32ACC, su3.SU3_C12_F32
MUL, MULADD = su3.SU3_EXPR_MUL, su3.SU3_EXPR_MULADD
DTYPE = {F64: torch.float64, F32: torch.float32, F16: torch.float16, C12: torch.float32}
P2, RAGGED, TINY = (16, 16, 16, 32), (7, 9, 11, 13), (1, 1, 1, 3)
P2F = (16, 16, 32, 32)  # planes of 2 MiB in single, 4 in double
P2H = (16, 32, 32, 32)  # of 2 MiB in half


def _field(dims, prec, seed):
    f = su3.field_tensor(dims, prec, su3.SU3_LAYOUT_SOA, 0)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    t = f.owner.view(DTYPE[prec])
    t.copy_(torch.randn(t.shape, generator=g, device="cuda").to(t.dtype))
    return f


@pytest.mark.parametrize("items", [
    [(P2, F64, MUL)], [(RAGGED, F64, MUL), (P2, F64, MUL), (TINY, C12, MUL)],
    [(TINY, C12, MUL), (P2F, C12, MUL), (RAGGED, C12, MUL)],
    [(P2F, F32, MUL), (RAGGED, F64, MUL), (P2F, F64, MUL)],
    [(RAGGED, F16, MUL), (P2H, F16, MUL), (TINY, F16, MULADD)],
    [(P2F, F32, MULADD), (P2, F64, MULADD), (RAGGED, F32, MUL)],
])
def test_ranges_equal_single_calls(items):
    s = torch.cuda.current_stream()
    su3.su3_launch_reset()
    exprs, zs, ops, want = [], [], [], []
    for i, (dims, prec, expr) in enumerate(items):
        o = [_field(dims, prec, 10 * i + k) for k in range(4 if expr == MULADD else 2)]
        y, z = _field(dims, prec, 10 * i + 9), _field(dims, prec, 10 * i + 9)
        su3.su3_fused_eval(y, expr, o, s)
        exprs.append(expr)
        zs.append(z)
        ops.append(o)
        want.append(y)
    b = su3.su3_batch_create(exprs, zs, ops, s)
    su3.su3_batch_launch(b, s)
    su3.su3_sync(s)
    for z, y in zip(zs, want):
        assert torch.equal(z.owner, y.owner)
