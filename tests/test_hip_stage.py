"""Host transfers through the pinned staging chunks: sizes around the direct
limit, a ragged last chunk, pinned sources, and several threads and streams at
once (more than there are staging sets)."""
import threading

import numpy as np
import pytest
import torch

from paper_1011_3318_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def W():
    from paper_1011_3318_amd import wcl
    return wcl


# bytes of the FP64 host field: 192 per site and rhs
#   10x10x20x20  7.7 MB, below the direct limit of 8 MiB
#   16x16x12x16  9.4 MB, three chunks, the last one ragged
#   9x11x13x17 x 3  12.6 MB, odd extents
@pytest.mark.parametrize("dims,nrhs", [((10, 10, 20, 20), 1), ((16, 16, 12, 16), 1), ((9, 11, 13, 17), 3)])
@pytest.mark.parametrize("pinned", [False, True])
def test_round_trip(W, dims, nrhs, pinned):
    ctx = W.Context(0)
    lat = W.Lattice(ctx, dims)
    psi = I.gaussian_source(dims, 4, nrhs=nrhs)
    if pinned:
        t = torch.empty(psi.size * 2, dtype=torch.float64, pin_memory=True)
        host = t.numpy().view(np.complex128).reshape(psi.shape)
        host[...] = psi
    else:
        host = psi
    dev = lat.pack(host, W.F64, nrhs)
    assert np.array_equal(lat.unpack(dev, W.F64, nrhs), psi)
    f32 = lat.unpack(lat.pack(host, W.F32, nrhs), W.F32, nrhs)
    assert np.array_equal(f32, psi.astype(np.complex64).astype(np.complex128))
    lat.close()
    ctx.close()


def test_many_threads_and_contexts(W):
    """Six threads, each with its own context, lattice and stream."""
    dims, bad = (16, 16, 12, 16), []
    psis = [I.gaussian_source(dims, 10 + k) for k in range(6)]

    def work(k):
        try:
            torch.cuda.set_device(0)
            st = torch.cuda.Stream()
            for rep in range(3):
                ctx = W.Context(0)
                lat = W.Lattice(ctx, dims)
                dev = lat.pack(psis[k], W.F64, stream=st)
                if not np.array_equal(lat.unpack(dev, W.F64, stream=st), psis[k]):
                    bad.append((k, rep))
                lat.close()
                ctx.close()
        except Exception as e:   # noqa: BLE001
            bad.append((k, repr(e)))

    th = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert bad == []


def test_kept_staging_gives_way(W):
    """The device block kept between transfers is not counted as in use and is
    given back when another allocation needs its room: a budget of exactly two
    resident lattices and one upload's staging is enough, as without it."""
    dims = (8, 8, 8, 8)
    V = I.volume(dims)
    # links 384 + 192 + 96, clover 576 + 288 + 148 bytes a site; staged FP64 links
    resident, staged = 1684 * V, 576 * V
    ctx = W.Context(0, hbm_budget=2 * resident + staged)
    U = I.random_gauge(dims, 0.5, 1)
    lats = []
    for k in range(2):
        lat = W.Lattice(ctx, dims)
        lat.upload_gauge(U)
        psi = I.gaussian_source(dims, 3 + k)
        assert np.array_equal(lat.unpack(lat.pack(psi, W.F64), W.F64), psi)
        lats.append(lat)
        assert ctx.bytes_in_use() <= (k + 1) * resident
    lats[0].upload_gauge(U)   # again, into the resident fields
    for lat in lats:
        lat.close()
    assert ctx.bytes_in_use() == 0
    ctx.close()


def test_per_thread_stream(W):
    """The per-thread default stream (handle 2), which names another stream in
    every host thread: an unpack of several chunks behind queued work returns
    that work's result."""
    dims, per_thread = (16, 16, 12, 16), 2
    ctx = W.Context(0)
    lat = W.Lattice(ctx, dims)
    lat.upload_gauge(I.random_gauge(dims, 0.5, 1))
    psi = I.gaussian_source(dims, 4)
    x, y = lat.pack(psi, W.F64), lat.zeros(W.F64)
    for _ in range(100):   # a few ms
        lat.apply_D(W.F64, 0.1, 1.0, x, y, stream=per_thread)
    lat.apply_D(W.F64, 0.126, 1.0, x, y, stream=per_thread)
    got = lat.unpack(y, W.F64, stream=per_thread)
    z = lat.apply_D(W.F64, 0.126, 1.0, lat.pack(psi, W.F64, stream=per_thread), lat.zeros(W.F64))
    torch.cuda.synchronize()
    assert np.array_equal(got, lat.unpack(z, W.F64))
    lat.close()
    ctx.close()
