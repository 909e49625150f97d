"""Tall slabs of the 3-D lane kernel at its largest block, 8^3 cells, on
forests large enough for the automatic height to give them (half blocks from
512 leaves, whole blocks from 1024), with a refined root: one step against the
oracle with periodic and outflow faces, and at degree 3 whole blocks against
the thread-per-cell kernel (the tolerances of the smaller forests' tests)."""
import numpy as np
import pytest

from paper_2502_12620_amd import workloads as W
from tests.gpu_helpers import make_pair, rel_diff, rel_diff_floored
from tests.test_gpu_parity import TOL, _cuda, _host, _physical_state

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _workload(p, roots, bc):
    w = W.Workload("tall", 3, p, 8, roots, (0.0,) * 3, tuple(float(r) for r in roots), (bc,) * 3, 2, W.IC_VORTEX,
                   [3.0, 1.0, 1.0, 0.5, 0.3, 2.0, 2.0], 1)
    w.initial_refinement = [lambda w_, keys: np.array([1 if k[0] == 5 else 0 for k in keys], np.int8)]
    return w


# (degree, roots, layers of a slab): 519 and 1027 leaves
@pytest.mark.parametrize("p,roots", [(3, (8, 8, 8)), (2, (17, 10, 6))])
@pytest.mark.parametrize("bc", [W.PERIODIC, W.OUTFLOW])
def test_tall_slabs_against_the_oracle(p, roots, bc):
    orc, gpu = make_pair(_workload(p, roots, bc))
    assert gpu.n_leaves >= (512 if p == 3 else 1024)
    u = _physical_state(orc, _workload(p, roots, bc), seed=p)
    ud, work, dt = _cuda(u), gpu.new_work(), torch.zeros(1, dtype=torch.float64, device="cuda")
    gpu.step(ud, work, dt, 0.1)
    orc.step(u, 0.1)
    assert rel_diff(_host(ud), u).max() <= TOL


def test_whole_blocks_at_degree_3_against_the_thread_per_cell_kernel():
    from paper_2502_12620_amd import dgamr as G

    w = _workload(3, (17, 10, 6), W.OUTFLOW)
    f = G.Forest(w.dim, w.degree, w.n_cell, w.roots, w.lo, w.hi, w.bc, w.max_level, w.gamma)
    f.adapt(w.initial_refinement[0](w, f.keys()), f.new_state())
    g = torch.Generator(device="cuda").manual_seed(3)
    u = 0.01 * torch.randn(f.state_shape(), dtype=torch.float64, device="cuda", generator=g)
    u[:, 0, 0] += 1.0
    u[:, 1, 0] += 0.3
    u[:, 4, 0] += 2.5
    work, dt, out = f.new_work(), torch.zeros(1, dtype=torch.float64, device="cuda"), []
    for variant in (0, 1):
        f.set_tuning(G.TUNE_STAGE_VARIANT, variant)
        us = u.clone()
        f.step(us, work, dt, 0.1)
        out.append(_host(us))
    assert rel_diff_floored(out[0], out[1], floor=1e-2).max() <= 1e-13
