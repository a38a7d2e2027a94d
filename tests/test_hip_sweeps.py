"""Edges of the domain sweeps: the split path's first MR step, which reads the
projection source in place (one step only, where it is also the last; ragged
domains; several right-hand sides), and the residual update's crossing hops of
the on-chip path on domains with a side of one site, antiperiodic directions and
right-hand sides in one launch; the binary16-operand sweeps on either side of the
grid size above which three domains share a CU."""
import numpy as np
import pytest

from helpers import rel_err
from oracle import Oracle
from paper_1011_3318_amd import inputs as I

pytestmark = pytest.mark.gpu

KAPPA, CSW = 0.124, 1.0


@pytest.fixture(scope="module")
def W():
    from paper_1011_3318_amd import wcl
    return wcl


# (dims, block, s): 384 extended sites (a half-empty second workgroup), 1296
# (16 sites in the last one), one domain spanning the whole lattice
# (these overlapping ones copy the source first, their x side being short), and
# two overlapping ones that read it in place
SPLIT = [((8, 4, 6, 4), (4, 2, 2, 4), 1), ((8, 8, 8, 8), (4, 4, 4, 4), 1), ((4, 6, 4, 4), (4, 6, 4, 4), 0),
         ((16, 4, 4, 4), (8, 4, 4, 4), 1), ((12, 4, 6, 8), (6, 4, 3, 4), 1)]


# the tolerances of the preconditioner's own tests: FP32 1e-4, FP16 storage 2e-2
@pytest.mark.parametrize("storage,tol", [(1, 1e-4), (2, 2e-2)])
@pytest.mark.parametrize("n_ras,nd", [(1, 1), (3, 1), (2, 2)])
@pytest.mark.parametrize("dims,block,s", SPLIT)
def test_split_first_step(W, dims, block, s, n_ras, nd, storage, tol):
    ctx = W.Context(0)
    U = I.random_gauge(dims, 0.5, 1)
    lat = W.Lattice(ctx, dims, (1, 1, 1, -1))
    lat.upload_gauge(U)
    r = I.gaussian_source(dims, 6, nrhs=2)
    ras = W.RasParams.make(block=block, s=s, n_ras=n_ras, n_dominv=nd, storage=storage, kernel=W.BLOCK_SPLIT)
    got = lat.unpack(lat.ras_precondition(ras, KAPPA, CSW, lat.pack(r, W.F32, 2), lat.empty(W.F32, 2), nrhs=2),
                     W.F32, 2)
    o = Oracle(dims, U, bc=(1, 1, 1, -1))
    for k in range(2):
        assert rel_err(got[k], o.ras(r[k], KAPPA, CSW, block, s, n_ras, nd)) <= tol
    lat.close()
    ctx.close()


# on chip: every site crosses in some direction; 240 sites of 256 lanes; one site
# per side in y; domains spanning x and t (no crossing there)
ONCHIP = [((4, 4, 4, 4), (2, 2, 2, 2)), ((8, 8, 6, 10), (4, 4, 3, 5)), ((6, 5, 4, 4), (3, 1, 4, 2)),
          ((4, 8, 8, 4), (4, 4, 4, 4))]


# binary16 operands and FP16 storage 2e-2, FP32 1e-4 (as above)
@pytest.mark.parametrize("storage,arith,tol", [(1, 0, 1e-4), (2, 0, 2e-2), (2, 1, 2e-2)])
@pytest.mark.parametrize("bc", [(1, 1, 1, 1), (-1, 1, -1, -1)])
@pytest.mark.parametrize("dims,block", ONCHIP)
def test_crossing_hops(W, dims, block, bc, storage, arith, tol):
    ctx = W.Context(0)
    U = I.random_gauge(dims, 0.5, 1)
    lat = W.Lattice(ctx, dims, bc)
    lat.upload_gauge(U)
    r = I.gaussian_source(dims, 6, nrhs=3)
    ras = W.RasParams.make(block=block, s=0, n_ras=3, n_dominv=3, storage=storage, arith=arith)
    got = lat.unpack(lat.ras_precondition(ras, KAPPA, CSW, lat.pack(r, W.F32, 3), lat.empty(W.F32, 3), nrhs=3),
                     W.F32, 3)
    o = Oracle(dims, U, bc=bc)
    for k in range(3):
        assert rel_err(got[k], o.ras(r[k], KAPPA, CSW, block, 0, 3, 3)) <= tol
    one = lat.unpack(lat.ras_precondition(ras, KAPPA, CSW, lat.pack(r[1], W.F32), lat.empty(W.F32)), W.F32)
    assert np.array_equal(one, got[1])
    lat.close()
    ctx.close()


# 256 domains per right-hand side: 256 and 512 workgroups run the form with two
# domains per CU, 768 the one with three; the bits must not depend on it
@pytest.mark.parametrize("n_ras,nd", [(1, 1), (2, 4), (3, 3)])
@pytest.mark.parametrize("bc", [(1, 1, 1, 1), (-1, 1, 1, -1)])
def test_domains_per_cu(W, bc, n_ras, nd):
    dims, block = (8, 8, 8, 8), (2, 2, 2, 2)
    ctx = W.Context(0)
    U = I.random_gauge(dims, 0.5, 1)
    lat = W.Lattice(ctx, dims, bc)
    lat.upload_gauge(U)
    r = I.gaussian_source(dims, 6, nrhs=3)
    ras = W.RasParams.make(block=block, s=0, n_ras=n_ras, n_dominv=nd, storage=W.F16, arith=W.ARITH_DOT2)

    def run(v, n):
        return lat.unpack(lat.ras_precondition(ras, KAPPA, CSW, lat.pack(v, W.F32, n), lat.empty(W.F32, n), nrhs=n),
                          W.F32, n)

    three = run(r, 3)
    assert np.array_equal(run(r[:2], 2), three[:2])
    for k in range(3):
        assert np.array_equal(np.asarray(run(r[k:k + 1], 1)).reshape(three[k].shape), three[k])
    o = Oracle(dims, U, bc=bc)
    assert rel_err(three[1], o.ras(r[1], KAPPA, CSW, block, 0, n_ras, nd)) <= 2e-2
    lat.close()
    ctx.close()
