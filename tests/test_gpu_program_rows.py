"""Matrix programs by rows: three waves hold the rows of 64 or 128 sites in
LDS.  Sizes on both sides of each choice of form (all workgroups resident or
not, four slots in single, AoS with and without a matrix result), ragged
tails, every mode of reading an operand, and fields updated in place, against
the oracle's evaluator.

Tolerance (absolute, per real entry): |got - want| <= 64 u (1 + max|want|),
u = 2^-53 or 2^-24: each expression is at most eight operations deep, each a
chain of at most six roundings over terms bounded by the largest value, plus
the rounding of the stored result."""
import numpy as np
import pytest
import torch

import oracle as O
import testgen
import paper_1710_09409_amd as su3

pytestmark = pytest.mark.gpu

M, R, C = su3.SU3_KIND_MATRIX, su3.SU3_KIND_REAL, su3.SU3_KIND_COMPLEX
F64, F32, C12 = su3.SU3_F64, su3.SU3_F32, su3.SU3_C12_F32
SOA, AOS = (su3.SU3_LAYOUT_SOA, 0), (su3.SU3_LAYOUT_AOS, 0)
A8, A64 = (su3.SU3_LAYOUT_AOSOA, 8), (su3.SU3_LAYOUT_AOSOA, 64)
FORCE = ("(a*b+c*d)*(a*c+b*d)+(a-b)*(c-d)", (M, M, M, M))
PATHS = ("a*b+c*d", (M, M, M, M))
PLAQUETTE = ("trace(a*b*adj(c)*adj(d))", (M, M, M, M))
MODES = ("c*adj(a*b) - transpose(conj(b))*a*d + trace(a*adj(b))*b - 0.5*i", (M, M, R, C))
SCALED = ("-(adj(a)*(c*b))*d + real(trace(b*a))", (M, M, R, C))
EIGHT = ("(a*b+c*d)*(e*f+g*h)", (M,) * 8)
TAIL = (3, 3, 3, 7)


def _make(dims, prec, kind, lay, host, s):
    if kind == M:
        f = su3.field_tensor(dims, prec, *lay)
    else:
        f = su3.scalar_tensor(dims, prec, lay[0], kind, lay[1])
    if host is not None:
        su3.su3_field_upload(f, host, s)
    return f


def _host(V, kind, k):
    if kind == M:
        return testgen.su3_field(V, field_id=500 + k)
    x = 3.0 * testgen.su3_field(V, field_id=510 + k).reshape(V, 18)
    return x[:, 0].copy() if kind == R else x[:, :2].copy()


@pytest.mark.parametrize("program,prec,lay,dims", [
    (MODES, F64, SOA, TAIL), (MODES, F32, SOA, TAIL), (MODES, C12, SOA, TAIL),
    (MODES, F64, AOS, TAIL), (MODES, F32, AOS, TAIL), (MODES, C12, AOS, TAIL),
    (MODES, F32, A8, TAIL), (MODES, C12, A64, TAIL),
    (SCALED, F64, A8, TAIL), (SCALED, F32, A64, TAIL), (SCALED, C12, AOS, TAIL),
    (PATHS, F32, SOA, (1, 1, 1, 1)), (PATHS, F64, AOS, (1, 1, 1, 64)),
    (PATHS, F32, A64, (1, 1, 5, 13)), (PATHS, F64, SOA, (1, 1, 5, 13)),
    # single: four slots fill the chip at 131072 sites
    (PATHS, F32, SOA, (16, 16, 16, 32)), (PATHS, F32, SOA, (16, 16, 16, 33)),
    # six slots: at 32768 sites in double, 65536 in single
    (FORCE, F64, SOA, (16, 16, 16, 8)), (FORCE, F64, A64, (16, 16, 9, 15)),
    (FORCE, F64, AOS, (16, 16, 9, 15)), (FORCE, F32, AOS, (16, 16, 17, 31)),
    (FORCE, F32, SOA, (16, 16, 16, 16)), (FORCE, C12, A64, (16, 16, 17, 16)),
    (PLAQUETTE, F64, AOS, TAIL), (PLAQUETTE, F64, SOA, (16, 16, 16, 17)),
    # more values than slots
    (EIGHT, F64, SOA, TAIL), (EIGHT, F32, AOS, TAIL),
])
def test_rows_parity(program, prec, lay, dims):
    s = torch.cuda.current_stream()
    V = testgen.volume(dims)
    text, kinds = program
    arith = F64 if prec == F64 else F32
    precs = [prec if k == M else arith for k in kinds]
    hosts = [_host(V, k, i) for i, k in enumerate(kinds)]
    fs = [_make(dims, p, k, lay, h, s) for p, k, h in zip(precs, kinds, hosts)]
    prog = su3.Program(text, kinds)
    rk = prog.info()["result_kind"]
    z = _make(dims, arith, rk, lay, None, s)
    z.owner.fill_(0x55)
    su3.su3_program_eval(prog, z, fs, s)
    got = su3.su3_field_download(z, s)
    q = [O.get().roundtrip(p, h) if k == M else h if p == F64 else
         h.astype(np.float32).astype(np.float64) for h, k, p in zip(hosts, kinds, precs)]
    want = O.get().eval_expr(text, q, [int(k) for k in kinds], V=V).reshape(got.shape)
    u = 2.0 ** -53 if arith == F64 else 2.0 ** -24
    assert np.max(np.abs(got - want)) <= 64 * u * (1 + np.max(np.abs(want)))
    # a copy by program has the same bytes, and neither writes the padding
    if rk == M:
        y = _make(dims, arith, rk, lay, None, s)
        y.owner.fill_(0x55)
        su3.su3_program_eval(su3.Program("a", (M,)), y, [z], s)
        assert torch.equal(y.owner, z.owner)


@pytest.mark.parametrize("prec", [F64, F32, C12])
@pytest.mark.parametrize("lay", [SOA, A64, AOS])
@pytest.mark.parametrize("text", ["adj(b)*a", "transpose(a)", "conj(a)*b*adj(a)"])
def test_rows_in_place(text, lay, prec):
    """The output is operand a: the same bits as into a field of its own."""
    s = torch.cuda.current_stream()
    dims = (9, 8, 5, 7)
    V = testgen.volume(dims)
    kinds = (M, M) if "b" in text else (M,)
    fs = [_make(dims, prec, k, lay, _host(V, k, i), s) for i, k in enumerate(kinds)]
    z = _make(dims, prec, M, lay, _host(V, M, 0), s)
    prog = su3.Program(text, kinds)
    su3.su3_program_eval(prog, z, fs, s)
    su3.su3_program_eval(prog, fs[0], fs, s)
    su3.su3_sync(s)
    assert torch.equal(z.owner, fs[0].owner)


@pytest.mark.parametrize("prec,dims,program", [
    (F64, (16, 16, 16, 32), PATHS), (F64, (16, 16, 16, 32), PLAQUETTE),
    (F32, (16, 16, 32, 32), PATHS), (F32, (16, 16, 32, 32), SCALED),  # by lanes, by rows
])
def test_ranges_per_xcd(prec, dims, program):
    """Planes of 2 MiB: workgroups in ranges by default, the bits of a launch
    that deals them one by one."""
    s = torch.cuda.current_stream()
    V = testgen.volume(dims)
    text, kinds = program
    fs = [_make(dims, prec, k, SOA, _host(V, k, i), s) for i, k in enumerate(kinds)]
    prog = su3.Program(text, kinds)
    rk = prog.info()["result_kind"]
    key = su3.SU3_EXPR_PROGRAM if rk == M else su3.SU3_EXPR_PROGRAM_SCALAR
    y, z = (_make(dims, prec, rk, SOA, None, s) for _ in range(2))
    su3.su3_launch_reset()
    default = su3.su3_launch_get(key, prec, SOA[0], 0, dims).as_dict()
    assert default["xcd_remap"] == 1
    su3.su3_program_eval(prog, z, fs, s)
    su3.su3_launch_set(key, prec, SOA[0], 0, dims, dict(default, xcd_remap=0))
    try:
        su3.su3_program_eval(prog, y, fs, s)
    finally:
        su3.su3_launch_reset()
    su3.su3_sync(s)
    assert torch.equal(y.owner, z.owner)
