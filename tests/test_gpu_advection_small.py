"""Scalar convection where its stage runs point by point in FP64 (degree 0,
and four-cell blocks at 2-D degree 1 and, up to 32768 leaves, 2) and right
past that line: steps and the residual against the oracle on hanging forests
in both modes, at the parity bar."""
import numpy as np
import pytest

from tests.gpu_helpers import rel_diff
from tests.test_gpu_advection import TOL, _cuda, _host, _pair, _state

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [(2, 0, 2, None), (2, 0, 6, None), (2, 0, 16, None), (2, 1, 2, None), (2, 2, 2, None), (2, 1, 4, None),
         (2, 2, 2, (182, 182)), (3, 0, 2, None), (3, 0, 6, None), (3, 1, 2, None)]


@pytest.mark.parametrize("dim,p,N,roots", CASES)
@pytest.mark.parametrize("hanging", [0, 1])
def test_convection_on_small_blocks(dim, p, N, roots, hanging):
    levels = 2 if roots or N > 6 else 3
    orc, gpu = _pair(dim, p, N, levels, hanging, roots=roots, hi=roots and tuple(float(r) for r in roots))
    if roots:
        assert gpu.n_leaves > 32768
    u = _state(orc, seed=dim + p + N)
    ud, guard, r = _cuda(u), gpu.new_guard(), gpu.new_residual()
    gpu.fill_guardcells(ud, guard)
    gpu.dg_residual(ud, guard, r)
    assert rel_diff(_host(r), orc.residual(u)).max() <= TOL
    work, dt = gpu.new_work(), torch.zeros(1, dtype=torch.float64, device="cuda")
    for _ in range(2):
        gpu.step(ud, work, dt, 0.1)
        orc.step(u, 0.1)
    assert np.isfinite(u).all()
    assert rel_diff(_host(ud), u).max() <= TOL
