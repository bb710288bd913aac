"""One batch launched on several streams in turn, eagerly and from a captured
graph: a persistent grid's launches share a ticket counter, and each still
writes every tile before its stream goes on."""
import pytest
import torch

import testgen
import paper_1710_09409_amd as su3
from gpu_util import upload

pytestmark = pytest.mark.gpu

F64, SOA = su3.SU3_F64, su3.SU3_LAYOUT_SOA


@pytest.mark.parametrize("persistent", [0, 2])
def test_streams_and_replays(persistent):
    s = torch.cuda.current_stream()
    lattices = [(16, 16, 16, 8), (7, 9, 5, 11), (12, 12, 12, 12)]
    hosts = [[testgen.su3_field(testgen.volume(d), field_id=60 + 2 * i + k) for k in (0, 1)]
             for i, d in enumerate(lattices)]
    ops = [[upload(d, F64, SOA, 0, h, s) for h in hs] for d, hs in zip(lattices, hosts)]
    zs = [su3.field_tensor(d, F64, SOA) for d in lattices]
    want = []
    for z, (x, y) in zip(zs, ops):
        z.owner.zero_()  # padding too
        su3.su3_mult(z, x, y, s)
        want.append(z.owner.clone())
    total = (sum(testgen.volume(d) for d in lattices), 1, 1, 1)
    key = su3.SU3_EXPR_BATCH + su3.SU3_EXPR_MUL
    cfg = su3.su3_launch_get(key, F64, SOA, 0, total)
    cfg.persistent, cfg.tile_sites, cfg.block = persistent, 64, 64
    su3.su3_launch_set(key, F64, SOA, 0, total, cfg)
    try:
        batch = su3.su3_batch_create([su3.SU3_EXPR_MUL] * len(zs), zs, ops, s)
    finally:
        su3.su3_launch_reset()
    streams = [torch.cuda.Stream() for _ in range(3)]
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        su3.su3_batch_launch(batch, torch.cuda.current_stream())
    for rep in range(6):
        # each stream reads the results of its own launch
        got = []
        for t in streams:
            with torch.cuda.stream(t):
                su3.su3_batch_launch(batch, t)
                got.append([z.owner.clone() for z in zs])
        torch.cuda.synchronize()
        for g in got:
            assert all(torch.equal(a, b) for a, b in zip(g, want)), rep
        for z in zs:
            z.owner.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(z.owner, w) for z, w in zip(zs, want)), rep
        for z in zs:
            z.owner.zero_()
        torch.cuda.synchronize()
    su3.su3_batch_destroy(batch)


@pytest.mark.parametrize("prec", [F64, su3.SU3_F32, su3.SU3_F16_F32ACC, su3.SU3_C12_F32],
                         ids=["f64", "f32", "f16", "c12"])
def test_every_entry(prec):
    """A batch launched, replayed from a graph and run without a handle writes
    every entry of every item, and nothing beyond them."""
    s = torch.cuda.current_stream()
    lattices = [(2, 3, 5, 7), (8, 8, 8, 8), (12, 12, 12, 13)]
    zs, ops, want = [], [], []
    for i, d in enumerate(lattices):
        hosts = [testgen.su3_field(testgen.volume(d), field_id=80 + 2 * i + k) for k in (0, 1)]
        x, y = (upload(d, prec, SOA, 0, h, s) for h in hosts)
        z = su3.field_tensor(d, prec, SOA)
        z.owner.fill_(0x55)
        su3.su3_mult(z, x, y, s)
        want.append(z.owner.clone())
        zs.append(z)
        ops.append([x, y])
    exprs = [su3.SU3_EXPR_MUL] * len(zs)
    batch = su3.su3_batch_create(exprs, zs, ops, s)
    graphs = [torch.cuda.CUDAGraph() for _ in range(2)]
    torch.cuda.synchronize()
    with torch.cuda.graph(graphs[0]):
        su3.su3_batch_launch(batch, torch.cuda.current_stream())
    with torch.cuda.graph(graphs[1]):
        su3.su3_batch_run(exprs, zs, ops, torch.cuda.current_stream())
    for go in (lambda: su3.su3_batch_launch(batch, s), graphs[0].replay, graphs[0].replay,
               graphs[1].replay, lambda: su3.su3_batch_run(exprs, zs, ops, s), graphs[1].replay):
        for z in zs:
            z.owner.fill_(0x55)
        torch.cuda.synchronize()
        go()
        torch.cuda.synchronize()
        assert all(torch.equal(z.owner, w) for z, w in zip(zs, want))
    su3.su3_batch_destroy(batch)
