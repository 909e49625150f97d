"""The limiter's quick acceptance (cells whose coefficient bounds already show
positive density and pressure skip the points) against the oracle, which looks
at every point: coefficients from no variation to far past the bounds in
neighbouring cells of a wave, densities and pressures at and below the
limiter's floor, non-finite cells, and kinetic energies that decide the
pressure.  A cell that needs no scaling keeps its bits; a scaled one is held
to the parity tests' bar."""
import numpy as np
import pytest

from paper_2502_12620_amd import workloads as W
from tests.gpu_helpers import make_pair, rel_diff
from tests.test_gpu_parity import TOL, _cuda, _forest, _host

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,p", [(2, 0), (2, 1), (2, 2), (2, 3), (3, 1), (3, 2), (3, 3)])
@pytest.mark.parametrize("mach", [0.0, 3.0])
def test_limiter_around_its_quick_acceptance(dim, p, mach):
    w = _forest(dim, p, 4, 2, bc=W.OUTFLOW)
    orc, gpu = make_pair(w)
    rng = np.random.default_rng(17 * dim + p)
    u = orc.project_ic(W.IC_UNIFORM, [1.0] + [0.0] * dim + [1.0])
    nl, nv, nb, nc = u.shape
    amp = 10.0 ** rng.uniform(-4, 0.7, size=(nl, 1, 1, nc))  # per cell: idle to heavily scaled
    u[:, :, 1:, :] = amp * rng.standard_normal((nl, nv, nb - 1, nc)) / max(1, nb - 1)
    u[:, 1, 0, :] = mach
    u[:, -1, 0, :] = 1.0 + 0.5 * mach * mach  # pressure decided by the difference
    tiny = rng.random((nl, nc)) < 0.05
    u[:, -1, 0, :] = np.where(tiny, 0.5 * mach * mach + 1e-13 * rng.uniform(-2, 4, (nl, nc)), u[:, -1, 0, :])
    thin = rng.random((nl, nc)) < (0.05 if mach == 0.0 else 0.0)  # densities at the floor, at rest on average
    for m in range(nb):
        u[:, 0, m, :] = np.where(thin, u[:, 0, m, :] * 1e-13, u[:, 0, m, :])
    ref = orc.limit(u.copy())
    ud = _cuda(u)
    gpu.limit_positivity(ud)
    got = _host(ud)
    assert rel_diff(got, ref).max() <= TOL
    same = (ref == u).all(axis=(1, 2))
    assert nb == 1 or (same.any() and not same.all())
    # a scaling factor of exactly one can come out as 1 - 2^-53 on one side only
    np.testing.assert_allclose(got.transpose(0, 3, 1, 2)[same], u.transpose(0, 3, 1, 2)[same], rtol=4e-16, atol=0)


def test_limiter_takes_the_points_for_non_finite_cells():
    w = _forest(2, 2, 4, 2, bc=W.OUTFLOW)
    orc, gpu = make_pair(w)
    u = orc.project_ic(W.IC_UNIFORM, [1.0, 0.0, 0.0, 1.0])
    u[0, 0, 1, 0] = np.nan
    u[0, 3, 2, 5] = np.inf
    u[1, 1, 0, 3] = -np.inf
    ref = orc.limit(u.copy())
    ud = _cuda(u)
    gpu.limit_positivity(ud)
    np.testing.assert_array_equal(np.isfinite(_host(ud)), np.isfinite(ref))
