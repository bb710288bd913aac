"""The end of a handle on borrowed memory while a stream is captured."""
import gc

import pytest
import torch

import testgen
import paper_1710_09409_amd as su3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["global", "thread_local", "relaxed"])
def test_capture_survives(mode):
    dims, s = (8, 8, 8, 8), torch.cuda.current_stream()
    host = testgen.su3_field(testgen.volume(dims), field_id=70)
    x, z = (su3.field_tensor(dims, su3.SU3_F64, su3.SU3_LAYOUT_SOA) for _ in range(2))
    su3.su3_field_upload(x, host, s)
    su3.su3_mult(z, x, x, s)
    want = z.owner.clone()
    memory, image = x.owner, z.owner
    gc.collect()  # the two handles are the last
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, capture_error_mode=mode):
        su3.su3_mult(z, x, x, torch.cuda.current_stream())
        su3.su3_field_free(x)
        su3.su3_field_free(z)
    for _ in range(3):
        image.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(image, want)
    assert memory.numel()
