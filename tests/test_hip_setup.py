"""The SU(3) test of a gauge upload (on the device, with the host deciding
close cases): which fields pass, the link that an error names, and that a
refused field leaves the resident one in place."""
import numpy as np
import pytest

from paper_1011_3318_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def W():
    from paper_1011_3318_amd import wcl
    return wcl


def _scaled(U, k, d):
    """Link k with its first row scaled: |U U^dag - 1| = 2 d."""
    V = U.reshape(-1, 3, 3).copy()
    V[k, 0] *= 1.0 + d
    return V


def _nan(U, k):
    V = U.reshape(-1, 3, 3).copy()
    V[k, 2, 2] = np.nan
    return V


def _swapped(U, k):
    V = U.reshape(-1, 3, 3).copy()
    V[k] = V[k][[1, 0, 2]]   # unitary, det = -1
    return V


# 64 links (less than a workgroup), 260 sites (a last workgroup with 16 links)
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 5, 13, 2)])
@pytest.mark.parametrize("last", [False, True])
def test_upload_su3_test(W, dims, last):
    ctx = W.Context(0)
    lat = W.Lattice(ctx, dims)
    U = I.random_gauge(dims, 0.5, 1)
    lat.upload_gauge(U)
    k = U.reshape(-1, 9).shape[0] - 1 if last else 0
    psi = I.gaussian_source(dims, 2)
    x, y = lat.pack(psi, W.F64), lat.empty(W.F64)
    before = lat.unpack(lat.apply_D(W.F64, 0.12, 1.0, x, y), W.F64)
    for bad in (_scaled(U, k, 0.55e-12), _scaled(U, k, 1e-3), _nan(U, k), _swapped(U, k), np.zeros_like(U),
                np.full_like(U, 1e200)):
        with pytest.raises(W.WclError) as e:
            lat.upload_gauge(bad)
        assert e.value.code == W.EUNITARITY
        first = k if bad.shape != U.shape else 0
        assert f"link {first} " in str(e.value)
    # the field before stays resident
    assert np.array_equal(lat.unpack(lat.apply_D(W.F64, 0.12, 1.0, x, y), W.F64), before)
    # within the tolerance: passed by the device alone, and by the host's second look
    for d in (0.2e-12, 0.47e-12):
        lat.upload_gauge(_scaled(U, k, d))
        got = lat.unpack(lat.apply_D(W.F64, 0.12, 1.0, x, y), W.F64)
        assert np.abs(got - before).max() < 1e-10
    lat.close()
    ctx.close()
