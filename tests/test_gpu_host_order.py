"""Upload and download with the conversion on the device: stored images byte
for byte the oracle's (numpy's for scalars), padding zero over old contents,
downloads bit for bit its unpacking -- below and above the size from which
the device converts, over several staging pieces, with infinities, signed
zeros, subnormals and values that round to a tie."""
import threading

import numpy as np
import pytest
import torch

import oracle
import testgen
import paper_1710_09409_amd as su3
from gpu_util import PRECS, PREC_NAMES

pytestmark = pytest.mark.gpu

SOA, AOSOA, AOS = su3.SU3_LAYOUT_SOA, su3.SU3_LAYOUT_AOSOA, su3.SU3_LAYOUT_AOS
LAYOUTS = ((AOS, 0), (SOA, 0), (AOSOA, 8), (AOSOA, 64))
# around 8192 stored reals of a matrix field; more than one 16 MiB piece
VOLUMES = ((1, 5, 7, 13), (4, 4, 29, 1), (9, 3, 13, 23), (33, 31, 29, 9))


def _values(V, seed):
    a = testgen.su3_field(V, field_id=seed)
    flat = a.reshape(-1)
    special = np.array([np.inf, -np.inf, -0.0, 5e-324, 2.0 ** -140, 2.0 ** -24, 65519.999, 1e300,
                        1.0 + 2.0 ** -24, 1.0 + 3 * 2.0 ** -11, 1.0 + 2.0 ** -11 + 2.0 ** -26])
    at = np.random.RandomState(seed).permutation(flat.size)[: special.size]
    flat[at] = special
    return a


@pytest.mark.parametrize("prec", PRECS, ids=lambda p: PREC_NAMES[p])
@pytest.mark.parametrize("dims", VOLUMES)
def test_matrix_images(prec, dims):
    s, orc = torch.cuda.current_stream(), oracle.get()
    V = testgen.volume(dims)
    host = _values(V, 7) if prec != su3.SU3_C12_F32 else testgen.su3_field(V, field_id=7)
    for layout, lanes in LAYOUTS:
        f = su3.field_tensor(dims, prec, layout, lanes)
        f.owner.fill_(0xAB)
        su3.su3_field_upload(f, host, s)
        want = orc.pack(host, prec, layout, lanes)
        assert np.array_equal(su3.su3_field_download_raw(f, s), np.asarray(want).view(np.uint8).ravel())
        got = su3.su3_field_download(f, s)
        assert np.array_equal(got.view(np.uint64),
                              orc.unpack(want, V, prec, layout, lanes).view(np.uint64))


@pytest.mark.parametrize("prec", PRECS, ids=lambda p: PREC_NAMES[p])
@pytest.mark.parametrize("dims,simd", [((8, 4, 6, 8), (1, 1, 2, 2)), ((4, 8, 12, 20), (2, 2, 2, 2)),
                                       ((6, 5, 7, 9), (1, 1, 1, 1))])
def test_virtual_node_images(prec, dims, simd):
    s, orc = torch.cuda.current_stream(), oracle.get()
    host = testgen.su3_field(testgen.volume(dims), field_id=8)
    f = su3.vnode_tensor(dims, prec, simd)
    su3.su3_field_upload(f, host, s)
    want = orc.vnode_pack(host, dims, simd, prec)
    assert np.array_equal(su3.su3_field_download_raw(f, s), want)
    # (the canonical data do not depend on the layout)
    canon = orc.unpack(orc.pack(host, prec, AOS), host.shape[0], prec, AOS)
    assert np.array_equal(su3.su3_field_download(f, s), canon)


@pytest.mark.parametrize("prec", [su3.SU3_F64, su3.SU3_F32])
@pytest.mark.parametrize("kind,per", [(su3.SU3_KIND_REAL, 1), (su3.SU3_KIND_COMPLEX, 2),
                                      (su3.SU3_KIND_SPINOR, 24)])
@pytest.mark.parametrize("dims", [(5, 7, 11, 13), (31, 30, 29, 31)])
def test_scalars_and_spinors(prec, kind, per, dims):
    s, V = torch.cuda.current_stream(), testgen.volume(dims)
    host = np.random.RandomState(3).standard_normal(V * per)
    stored = host if prec == su3.SU3_F64 else host.astype(np.float32)
    for layout, lanes, L in ((AOS, 0, 1), (SOA, 0, -(-V // 64) * 64), (AOSOA, 16, 16)):
        if kind == su3.SU3_KIND_SPINOR:
            f = su3.spinor_tensor(dims, prec, layout, lanes)
        else:
            f = su3.scalar_tensor(dims, prec, layout, kind, lanes)
        f.owner.fill_(0xAB)
        su3.su3_field_upload(f, host, s)
        E, c = (12, 2) if kind == su3.SU3_KIND_SPINOR else (1, per)
        blocks = -(-V // L)
        image = np.zeros((blocks * L, E, c), stored.dtype)
        image[:V] = stored.reshape(V, E, c)
        image = image.reshape(blocks, L, E, c).transpose(0, 2, 1, 3).copy().view(np.uint8).ravel()
        assert np.array_equal(su3.su3_field_download_raw(f, s), image)
        assert np.array_equal(su3.su3_field_download(f, s).ravel(), stored.astype(np.float64))


def test_threads_and_streams():
    """Transfers of several threads, each on a stream of its own, at once."""
    dims = (20, 20, 20, 18)
    V = testgen.volume(dims)
    hosts = [testgen.su3_field(V, field_id=40 + k) for k in range(6)]
    bad = []

    def work(k):
        s = torch.cuda.Stream()
        for _ in range(3):
            f = su3.field_tensor(dims, su3.SU3_F64, (SOA, AOSOA)[k % 2], 32 * (k % 2))
            torch.cuda.synchronize()
            su3.su3_field_upload(f, hosts[k], s)
            if not np.array_equal(su3.su3_field_download(f, s), hosts[k]):
                bad.append(k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
