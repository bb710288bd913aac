"""Transfers on both sides of the size from which a field is converted on the
device: one site below it, at it and one above, the stored field and the way
back are those of the host's conversion (exact in double, rounded as declared
otherwise)."""
import numpy as np
import pytest
import torch

import oracle as O
import testgen
import paper_1710_09409_amd as su3

pytestmark = pytest.mark.gpu

F64, F32, F16, C12 = su3.SU3_F64, su3.SU3_F32, su3.SU3_F16_F32ACC, su3.SU3_C12_F32
DTYPE = {F64: torch.float64, F32: torch.float32, F16: torch.float16, C12: torch.float32}


@pytest.mark.parametrize("layout,lanes", [(su3.SU3_LAYOUT_SOA, 0), (su3.SU3_LAYOUT_AOS, 0),
                                          (su3.SU3_LAYOUT_AOSOA, 16)], ids=["soa", "aos", "aosoa16"])
@pytest.mark.parametrize("prec,line", [(F64, 512), (F32, 550), (F16, 224), (C12, 960)],
                         ids=["f64", "f32", "f16", "c12"])
def test_sites_at_the_line(prec, line, layout, lanes):
    s = torch.cuda.current_stream()
    for V in (line - 1, line, line + 1):
        dims = (V, 1, 1, 1)
        host = testgen.su3_field(V, field_id=testgen.FID_X)
        want = O.get().roundtrip(prec, host)
        f = su3.field_tensor(dims, prec, layout, lanes)
        su3.su3_field_upload(f, host, s)
        su3.su3_sync(s)
        entries = 6 if prec == C12 else 9
        raw = f.owner.view(DTYPE[prec]).cpu().numpy().astype(np.float64).ravel()
        block = {su3.SU3_LAYOUT_SOA: (V + 63) // 64 * 64, su3.SU3_LAYOUT_AOS: 1}.get(layout, lanes)
        site = np.arange(V)[:, None]
        at = ((site // block) * entries + np.arange(entries)) * 2 * block + site % block * 2
        stored = host.reshape(V, 9, 2)[:, :entries]
        if prec != F64:
            stored = stored.astype(np.float32)
        if prec == F16:  # by way of single, the declared rounding of half storage
            stored = stored.astype(np.float16)
        assert np.array_equal(raw[at], stored[..., 0]), V
        assert np.array_equal(raw[at + 1], stored[..., 1]), V
        got = su3.su3_field_download(f, s)
        assert np.array_equal(got.reshape(-1), np.asarray(want).reshape(-1)), V
