"""AoS calls at the edges of their LDS tiles: volumes around one and two
workgroups' tiles, the last tile partial or whole, against the oracle; in
place too, and with every store form the kernel is compiled for."""
import numpy as np
import pytest
import torch

import paper_1710_09409_amd as su3
from gpu_util import (PRECS, PREC_NAMES, assert_parity, exprs_for, operands, reference, run_expr,
                      upload)

pytestmark = pytest.mark.gpu

AOS = su3.SU3_LAYOUT_AOS


@pytest.mark.parametrize("prec", PRECS, ids=lambda p: PREC_NAMES[p])
@pytest.mark.parametrize("V", [1, 63, 64, 65, 127, 128, 129, 1000])
def test_tile_edges(prec, V):
    dims = (V, 1, 1, 1)
    for expr in exprs_for(prec):
        host = operands(dims, expr)
        want = reference(prec, expr, host)
        got, _ = run_expr(dims, prec, AOS, 0, expr, host)
        assert_parity(prec, expr, got, want, f"default, expr {expr}")
        for block, nt in ((64, 0), (64, 7), (128, 2), (128, 3)):
            if block == 128 and prec == su3.SU3_F64 and expr == su3.SU3_EXPR_MULADD:
                continue  # its tiles exceed the staging limit
            cfg = su3.su3_launch_get(expr, prec, AOS, 0, dims)
            cfg.lds_stage, cfg.block, cfg.nontemporal, cfg.occupancy = 1, block, nt, 0
            su3.su3_launch_set(expr, prec, AOS, 0, dims, cfg)
            try:
                again, _ = run_expr(dims, prec, AOS, 0, expr, host)
            finally:
                su3.su3_launch_reset()
            assert np.array_equal(again, got), (expr, block, nt)


@pytest.mark.parametrize("V", [64, 200])
def test_in_place(V):
    dims, s = (V, 1, 1, 1), torch.cuda.current_stream()
    for prec in PRECS:
        host = operands(dims, su3.SU3_EXPR_MUL)
        x, y = (upload(dims, prec, AOS, 0, h, s) for h in host)
        su3.su3_mult(x, x, y, s)
        assert_parity(prec, su3.SU3_EXPR_MUL, su3.su3_field_download(x, s),
                      reference(prec, su3.SU3_EXPR_MUL, host), f"in place, prec {prec}")
