"""Shifted products and copies with each XCD on a range of workgroups: bit for
bit the launch without, at volumes a workgroup and eight do and do not divide,
and by default where entry planes are 2 to 16 MiB apart."""
import pytest
import torch

import paper_1710_09409_amd as su3
from test_gpu_default_launch import AOS, C12, F16, F32, F64, PLAIN, SOA, _fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,layout,dims,remap", [
    (F64, SOA, (16, 16, 16, 32), 1), (F32, SOA, (16, 16, 32, 32), 1),
    (C12, SOA, (16, 16, 32, 32), 1), (F16, SOA, (16, 32, 32, 32), None),
    (F64, SOA, (7, 9, 11, 13), 0), (F32, AOS, (5, 6, 7, 9), 0), (F16, SOA, (1, 3, 5, 7), 0),
])
@pytest.mark.parametrize("product", [True, False])
def test_shift_ranges(product, prec, layout, dims, remap):
    key = su3.SU3_EXPR_MUL_SHIFTED if product else su3.SU3_EXPR_CSHIFT
    x, y, z = _fields(3, dims, prec, layout, 0)
    s = torch.cuda.current_stream()

    def run(cfg):
        su3.su3_launch_reset()
        if cfg:
            su3.su3_launch_set(key, prec, layout, 0, dims, cfg)
        try:
            z.owner.fill_(0x33)
            if product:
                su3.su3_mult_shifted(z, x, y, 2, -1, s)
            else:
                su3.su3_cshift(z, y, 2, -1, s)
        finally:
            su3.su3_launch_reset()
        return z.owner.clone()

    want = run(dict(PLAIN, schedule=int(layout != AOS)))
    default = su3.su3_launch_get(key, prec, layout, 0, dims).as_dict()
    assert remap is None or default["xcd_remap"] == remap
    assert torch.equal(run(None), want)
    for block in (64, 256):
        cfg = dict(PLAIN, schedule=int(layout != AOS), block=block, xcd_remap=1)
        assert torch.equal(run(cfg), want)
