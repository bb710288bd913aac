"""Programs without matrix values: lanes of a wave take consecutive vectors of
16 bytes of a complex field, two vectors each.  Volumes around a vector, a
wave and a workgroup, real and complex operands mixed, both results.

Tolerance (absolute): |got - want| <= 64 u (1 + max|want|), u = 2^-53 or
2^-24: at most eight operations deep, each a chain of at most six roundings
over terms bounded by the largest value, plus the rounding of the result."""
import numpy as np
import pytest
import torch

import oracle as O
import testgen
import paper_1710_09409_amd as su3

pytestmark = pytest.mark.gpu

R, C = su3.SU3_KIND_REAL, su3.SU3_KIND_COMPLEX


@pytest.mark.parametrize("dims", [(1, 1, 1, 1), (1, 1, 1, 63), (1, 1, 1, 127), (1, 1, 1, 128),
                                  (1, 1, 3, 43), (1, 1, 3, 85), (1, 1, 1, 257), (1, 3, 11, 31),
                                  (1, 1, 25, 41), (5, 7, 9, 13)])
@pytest.mark.parametrize("prec", [su3.SU3_F64, su3.SU3_F32])
def test_scalar_programs(prec, dims):
    s = torch.cuda.current_stream()
    V = testgen.volume(dims)
    for text, kinds in [("a*conj(b)+a", (C, C)), ("c*a - imag(b)*conj(a) + 2*i", (C, C, R)),
                        ("real(a*b) - c", (C, C, R))]:
        hosts, fs = [], []
        for k, kind in enumerate(kinds):
            x = 3.0 * testgen.su3_field(V, field_id=530 + k).reshape(V, 18)
            hosts.append(x[:, 0].copy() if kind == R else x[:, :2].copy())
            fs.append(su3.scalar_tensor(dims, prec, su3.SU3_LAYOUT_SOA, kind, 0))
            su3.su3_field_upload(fs[-1], hosts[-1], s)
        if prec == su3.SU3_F32:
            hosts = [h.astype(np.float32).astype(np.float64) for h in hosts]
        prog = su3.Program(text, kinds)
        z = su3.scalar_tensor(dims, prec, su3.SU3_LAYOUT_SOA, prog.info()["result_kind"], 0)
        z.owner.fill_(0x55)
        su3.su3_program_eval(prog, z, fs, s)
        got = su3.su3_field_download(z, s)
        want = O.get().eval_expr(text, hosts, [int(k) for k in kinds], V=V).reshape(got.shape)
        u = 2.0 ** -53 if prec == su3.SU3_F64 else 2.0 ** -24
        assert np.max(np.abs(got - want)) <= 64 * u * (1 + np.max(np.abs(want)))
        used = got.size * (8 if prec == su3.SU3_F64 else 4)
        assert np.all(su3.su3_field_download_raw(z, s)[used:] == 0x55)  # padding left alone
