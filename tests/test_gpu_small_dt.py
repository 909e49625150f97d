"""The time step of small forests (one workgroup over all cells) against the
oracle: a single leaf, partial waves, and forests on either side of the size
where one workgroup per leaf takes over.  The maximum does not depend on the
order and each cell's rate is a dozen operations: the bar is the parity
tests' 1e-14 of dt."""
import numpy as np
import pytest

import oracle as O
from paper_2502_12620_amd import workloads as W
from tests.gpu_helpers import make_pair
from tests.test_gpu_parity import _cuda, _host, _physical_state

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (dim, N, roots): 4, 36, 2000, 2048 and 2112 cells; 8, 216, 2048 and 2560
CASES = [(2, 2, (1, 1)), (2, 6, (1, 1)), (2, 10, (5, 4)), (2, 8, (8, 4)), (2, 8, (11, 3)),
         (3, 2, (1, 1, 1)), (3, 6, (1, 1, 1)), (3, 8, (2, 2, 1)), (3, 8, (5, 1, 1))]


@pytest.mark.parametrize("dim,N,roots", CASES)
@pytest.mark.parametrize("p", [0, 2])
def test_dt_of_small_forests(dim, N, roots, p):
    w = W.Workload("s", dim, p, N, roots, (0.0,) * dim, tuple(float(r) for r in roots), (0,) * dim, 1, W.IC_VORTEX,
                   [3.0, 1.0, 1.0, 0.5, 0.3, 2.0, 2.0], 1)
    w.initial_refinement = []
    orc, gpu = make_pair(w)
    u = _physical_state(orc, w, seed=N + p)
    for where in (0, -1):  # the fastest cell first, then last
        v = u.copy()
        v[where, 1, 0, where] += 3.0
        v[where, -1, 0, where] += 20.0
        ud, work, dt = _cuda(v), gpu.new_work(), torch.zeros(1, dtype=torch.float64, device="cuda")
        gpu.step(ud, work, dt, 0.1)
        ref = orc.dt(v, 0.1)
        assert abs(_host(dt)[0] - ref) <= 1e-14 * ref
