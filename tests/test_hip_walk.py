"""Launches that walk the lattice's tiles in another order than they are
stored (columns cut in x or y), launches on small lattices, and the parity-split fields of the even-odd
operator with and without room for the split links, against the oracle."""
import numpy as np
import pytest

from helpers import rel_err
from oracle import Oracle
from paper_1011_3318_amd import inputs as I

pytestmark = pytest.mark.gpu

# column cross-section and the 64-site tiles of one column at one t:
#   24x8x8x4    8x8x8, 8 tiles (4 of a half field), three columns in x
#   12x12x4x6   4x4x4, 1 tile; half fields: storage order
#   12x20x16x4  4x4x8, 2 tiles (1 of a half field), two z ranges of 15 columns
#   10x6x4x6    2x2x4: storage order throughout
DIMS = [(24, 8, 8, 4), (12, 12, 4, 6), (12, 20, 16, 4), (10, 6, 4, 6)]
BC = (1, 1, 1, -1)


@pytest.fixture(scope="module")
def W():
    from paper_1011_3318_amd import wcl
    return wcl


# the tolerances of the D-apply's and the Schur operator's own tests
@pytest.mark.parametrize("dims", DIMS)
def test_walk_matches_oracle(W, dims):
    ctx = W.Context(0)
    U = I.random_gauge(dims, 0.5, 1)
    lat = W.Lattice(ctx, dims, BC)
    lat.upload_gauge(U)
    o = Oracle(dims, U, bc=BC)
    psi = I.gaussian_source(dims, 4, nrhs=2)
    kappa, csw = 0.126, 1.3
    ref = [o.apply_D(psi[k], kappa, csw) for k in range(2)]
    for prec, tol in ((W.F64, 1e-13), (W.F32, 1e-5), (W.F16, 2e-3)):
        out = lat.empty(prec, 2)
        got = lat.unpack(lat.apply_D(prec, kappa, csw, lat.pack(psi, prec, 2), out, nrhs=2), prec, 2)
        assert max(rel_err(got[k], ref[k]) for k in range(2)) <= tol
    for prec, tol in ((W.F64, 1e-13), (W.F32, 1e-5)):
        out = lat.empty(prec, 2)
        got = lat.unpack(lat.apply_schur(prec, kappa, csw, lat.pack(psi, prec, 2), out, nrhs=2), prec, 2)
        assert max(rel_err(got[k], o.apply_schur(psi[k], kappa, csw)) for k in range(2)) <= tol
    lat.close()
    ctx.close()


# launches with one wavefront per direction: less than a tile, a last tile of
# 4 sites, the largest lattice that takes them, and the next that does not
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 5, 13, 2), (8, 8, 8, 8), (8, 9, 8, 8)])
def test_small_launches(W, dims):
    ctx = W.Context(0)
    U = I.random_gauge(dims, 0.5, 1)
    lat = W.Lattice(ctx, dims, BC)
    lat.upload_gauge(U)
    o = Oracle(dims, U, bc=BC)
    psi = I.gaussian_source(dims, 4, nrhs=3)
    ref = [o.apply_D(psi[k], 0.126, 1.3) for k in range(3)]
    for prec, tol in ((W.F64, 1e-13), (W.F32, 1e-5), (W.F16, 2e-3)):
        got = lat.unpack(lat.apply_D(prec, 0.126, 1.3, lat.pack(psi, prec, 3), lat.empty(prec, 3), nrhs=3), prec, 3)
        assert max(rel_err(got[k], ref[k]) for k in range(3)) <= tol
        one = lat.unpack(lat.apply_D(prec, 0.126, 1.3, lat.pack(psi[2], prec), lat.empty(prec)), prec)
        assert np.array_equal(one, got[2])
    # the dot-product epilogue and the residual: a plain solve
    phi = lat.empty(W.F64)
    rc, st = lat.solve_bicgstab_f64(1e-11, 500, 0.11, 1.0, lat.pack(psi[0], W.F64), phi)
    sol = lat.unpack(phi, W.F64)
    assert rel_err(o.apply_D(sol, 0.11, 1.0), psi[0]) <= 1e-10
    lat.close()
    ctx.close()


# groups of right-hand sides with a smaller last one (7 = 4 + 3, 13 = 5 + 5 + 3),
# in the exchange layout (16x16x8x6: halved z ranges in FP64), with columns cut
# in x (24x8x8x10) and in storage order (10x6x14x6); all above 4096 sites
@pytest.mark.parametrize("dims", [(16, 16, 8, 6), (24, 8, 8, 10), (10, 6, 14, 6)])
@pytest.mark.parametrize("nrhs", [7, 13])
def test_rhs_groups(W, dims, nrhs):
    ctx = W.Context(0)
    lat = W.Lattice(ctx, dims, BC)
    lat.upload_gauge(I.random_gauge(dims, 0.5, 1))
    psi = I.gaussian_source(dims, 4, nrhs=nrhs)
    for prec in (W.F64, W.F32, W.F16):
        ops = [lat.apply_D] if prec == W.F16 else [lat.apply_D, lat.apply_schur]
        x = lat.pack(psi, prec, nrhs)
        for op in ops:
            many = lat.unpack(op(prec, 0.126, 1.3, x, lat.empty(prec, nrhs), nrhs=nrhs), prec, nrhs)
            for k in (0, 3, 4, 5, nrhs - 1):
                one = op(prec, 0.126, 1.3, lat.pack(psi[k], prec), lat.empty(prec))
                assert np.array_equal(lat.unpack(one, prec), many[k])
    lat.close()
    ctx.close()


@pytest.mark.parametrize("dims", DIMS[:2])
def test_schur_without_room_for_split_links(W, dims):
    """A budget that holds the call's own buffers but not the extra copy of
    the links: the same result, bit for bit."""
    U = I.random_gauge(dims, 0.5, 1)
    psi = I.gaussian_source(dims, 4)
    got, used = {}, {}
    for prec in (W.F64, W.F32):
        for budget in (0, 1):
            # 1680 bytes a site resident (links and clover), up to 672 for the
            # call, 192 staged by unpack
            ctx = W.Context(0, hbm_budget=budget * (2700 * I.volume(dims) + 65536))
            lat = W.Lattice(ctx, dims, BC)
            lat.upload_gauge(U)
            out = lat.empty(prec)
            lat.apply_schur(prec, 0.126, 1.3, lat.pack(psi, prec), out)
            got[prec, budget] = lat.unpack(out, prec)
            used[prec, budget] = ctx.bytes_in_use()
            lat.close()
            ctx.close()
        assert used[prec, 1] < used[prec, 0]
        assert np.array_equal(got[prec, 0], got[prec, 1])


# t extents that let cut columns be walked side by side (more than 10 t slices
# of all z ranges), just past the rule and beside it: 24x8x8 has one z range,
# 12x20x16 two
@pytest.mark.parametrize("dims", [(24, 8, 8, 10), (24, 8, 8, 12), (12, 12, 4, 14), (12, 20, 16, 6)])
def test_walk_side_by_side(W, dims):
    test_walk_matches_oracle(W, dims)


# batches on small lattices: groups of right-hand sides (7 = 4 + 3, 13 = 5 + 5 + 3)
# and, in FP16, the last count of tiles below the pipelined form's and the first above
# (1400): 2x5x13x2 has 5 tiles, the last of 4 sites
@pytest.mark.parametrize("dims,nrhs", [((8, 8, 8, 8), 7), ((8, 8, 8, 8), 13), ((8, 8, 8, 8), 21), ((8, 8, 8, 8), 22),
                                       ((2, 5, 13, 2), 280), ((2, 5, 13, 2), 281), ((15, 13, 7, 3), 22)])
def test_small_batches(W, dims, nrhs):
    ctx = W.Context(0)
    U = I.random_gauge(dims, 0.5, 1)
    lat = W.Lattice(ctx, dims, BC)
    lat.upload_gauge(U)
    o = Oracle(dims, U, bc=BC)
    psi = I.gaussian_source(dims, 4, nrhs=nrhs)
    for prec, tol in ((W.F64, 1e-13), (W.F32, 1e-5), (W.F16, 2e-3)):
        many = lat.unpack(lat.apply_D(prec, 0.126, 1.3, lat.pack(psi, prec, nrhs), lat.empty(prec, nrhs), nrhs=nrhs),
                          prec, nrhs)
        assert rel_err(many[nrhs - 1], o.apply_D(psi[nrhs - 1], 0.126, 1.3)) <= tol
        for k in range(nrhs) if nrhs < 30 else (0, 3, 4, 5, 6, nrhs // 2, nrhs - 1):
            one = lat.apply_D(prec, 0.126, 1.3, lat.pack(psi[k], prec), lat.empty(prec))
            assert np.array_equal(lat.unpack(one, prec), many[k]), (prec, k)
    lat.close()
    ctx.close()
