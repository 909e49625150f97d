"""Which 2-D stage kernel runs, by the bits of the state after two steps (the
two kernels round differently).  DGAMR_TUNE_VAR_SPLIT_MAX_CELLS decides between the 2-D stage kernels at
every block size.  Automatically, conservative forests with hanging faces
keep the lane kernel (where a mortar face costs a quarter of the time) up to
larger counts than forests without."""
import numpy as np
import pytest

from tests.gpu_helpers import make_pair
from tests.test_gpu_parity import _cuda, _forest, _physical_state

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [2, 4, 6])
def test_cell_limit_of_the_2d_lane_kernel(N):
    from paper_2502_12620_amd import dgamr as G

    w = _forest(2, 2, N, 2)
    orc, gpu = make_pair(w)
    u = _physical_state(orc, w, seed=N)
    cells = gpu.n_leaves * N * N

    def steps(knob, value):
        gpu.set_tuning(G.TUNE_STAGE_VARIANT, -1)
        gpu.set_tuning(knob, value)
        ud, work, dt = _cuda(u), gpu.new_work(), torch.zeros(1, dtype=torch.float64, device="cuda")
        for _ in range(2):
            gpu.step(ud, work, dt, 0.1)
        return ud

    lanes, cell = steps(G.TUNE_STAGE_VARIANT, 0), steps(G.TUNE_STAGE_VARIANT, 1)
    assert not torch.equal(lanes, cell)
    assert torch.equal(steps(G.TUNE_VAR_SPLIT_MAX_CELLS, 0), cell)
    assert torch.equal(steps(G.TUNE_VAR_SPLIT_MAX_CELLS, cells - 1), cell)
    assert torch.equal(steps(G.TUNE_VAR_SPLIT_MAX_CELLS, cells), lanes)


# (degree, N, roots, kernel with a hanging face, kernel without)
MORTAR = [(2, 8, (25, 25), 0, 1), (3, 16, (21, 20), 0, 1), (1, 16, (13, 13), 0, 1), (1, 16, (17, 16), 1, 1),
          (0, 16, (13, 13), 1, 1)]


@pytest.mark.parametrize("p,N,roots,with_mortar,without", MORTAR)
@pytest.mark.parametrize("refined", [False, True])
def test_kernel_of_conservative_forests(p, N, roots, with_mortar, without, refined):
    from paper_2502_12620_amd import dgamr as G

    f = G.Forest(2, p, N, roots, (0.0, 0.0), tuple(map(float, roots)), (0, 0), 2, 1.4, hanging=G.HANG_CONSERVATIVE)
    if refined:
        flags = np.zeros(f.n_leaves, np.int8)
        flags[7] = 1
        f.adapt(flags, f.new_state())
    g = torch.Generator(device="cuda").manual_seed(p)
    u = 0.01 * torch.randn(f.state_shape(), dtype=torch.float64, device="cuda", generator=g)
    u[:, 0, 0] += 1.0
    u[:, 3, 0] += 2.5
    work, dt = f.new_work(), torch.zeros(1, dtype=torch.float64, device="cuda")
    guard, out = f.new_guard(), {}
    f.fill_guardcells(u, guard)
    for variant in (-1, 0, 1):
        f.set_tuning(G.TUNE_STAGE_VARIANT, variant)
        us, r = u.clone(), f.new_residual()
        for _ in range(2):
            f.step(us, work, dt, 0.1)
        f.dg_residual(u, guard, r)
        out[variant] = us, r
    want = with_mortar if refined else without
    for k in range(2):
        assert torch.equal(out[-1][k], out[want][k])
        if p > 0:
            assert not torch.equal(out[-1][k], out[1 - want][k])
