"""Traces of negatives and conjugates bit for bit: each term changes its sign
before the sum, so the zero of a sum that cancels keeps its sign."""
import numpy as np
import pytest
import torch

import paper_1710_09409_amd as su3

pytestmark = pytest.mark.gpu

M, C = su3.SU3_KIND_MATRIX, su3.SU3_KIND_COMPLEX


@pytest.mark.parametrize("prec", [su3.SU3_F64, su3.SU3_F32], ids=["f64", "f32"])
@pytest.mark.parametrize("layout,lanes", [(su3.SU3_LAYOUT_AOS, 0), (su3.SU3_LAYOUT_SOA, 0),
                                          (su3.SU3_LAYOUT_AOSOA, 8)])
def test_zero_signs(prec, layout, lanes):
    s, dims = torch.cuda.current_stream(), (5, 7, 4, 9)
    V = 5 * 7 * 4 * 9
    host = np.random.RandomState(5).randint(-1, 2, (V, 3, 3, 2)).astype(np.float64)
    a = su3.field_tensor(dims, prec, layout, lanes)
    su3.su3_field_upload(a, host, s)
    z = su3.scalar_tensor(dims, prec, layout, C, lanes)
    diag = host[:, [0, 1, 2], [0, 1, 2], :]

    def trace(d):
        return (d[:, 0] + d[:, 1]) + d[:, 2]

    conj = np.array([1.0, -1.0])
    for text, want in (("trace(-a)", trace(-diag)), ("trace(conj(a))", trace(diag * conj)),
                       ("trace(adj(-a))", trace(-(diag * conj))),
                       ("trace(transpose(a))", trace(diag)), ("-trace(a)", -trace(diag)),
                       ("conj(trace(a))", trace(diag) * conj)):
        su3.su3_program_eval(su3.Program(text, [M]), z, [a], s)
        su3.su3_sync(s)
        got = su3.su3_field_download(z, s).reshape(V, 2)
        assert np.array_equal(got.view(np.uint64), want.view(np.uint64)), text
