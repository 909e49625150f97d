"""Workgroups of the 3-D lane kernel whose last item slots repeat the last
item (leaves and slabs that do not fill the groups): the CFL rate folded into
the last stage of a step, which stores the state in place, is that of the
state it stored.  The fastest cells lie in the last leaf and get faster, so
that a rate taken from a repeated item's mixture of old and new state would
win the maximum.  dt of dgamr_run and of a captured run against the separate
rate reduction of the same states (dgamr_step): a dozen operations per cell on
states that agree to rounding, 1e-13."""
import numpy as np
import pytest

from paper_2502_12620_amd import workloads as W
from tests.gpu_helpers import rel_diff_floored
from tests.test_gpu_parity import _cuda, _host

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (degree, N, roots): groups of four items at N = 2 (two of one-layer slabs at
# 1, 3 and 5 leaves: 2 of 4, 6 of 8 and 10 of 12), of two at N = 4 and 8 (from
# 1025 leaves whole-leaf items: 1025 of 1026)
CASES = [(2, 2, (1, 1, 1)), (2, 2, (3, 1, 1)), (3, 2, (5, 1, 1)), (2, 4, (41, 25, 1)), (3, 4, (41, 25, 1)),
         (2, 8, (41, 25, 1)), (3, 8, (41, 25, 1))]


@pytest.mark.parametrize("p,N,roots", CASES)
@pytest.mark.parametrize("captured", [False, True])
def test_rate_of_partly_filled_groups(p, N, roots, captured):
    from paper_2502_12620_amd import dgamr as G

    f = G.Forest(3, p, N, roots, (0.0,) * 3, tuple(float(r) for r in roots), (W.PERIODIC,) * 3, 1, 1.4)
    u = np.zeros(f.state_shape())
    u[:, 0, 0] = 1.0
    u[:, 4, 0] = 2.5
    back = np.arange(N ** 3) % N >= N // 2
    vx, pr = np.where(back, 5.0, 1.0), np.where(back, 1.0, 4.0)
    u[-1, 1, 0] = vx
    u[-1, 4, 0] = 2.5 * pr + 0.5 * vx ** 2
    ur, us = _cuda(u), _cuda(u)
    work, dt_r, dt_s = f.new_work(), *(torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2))
    dts = []
    for _ in range(3):
        f.step(us, work, dt_s, 0.05)
        dts.append(_host(dt_s)[0])
    assert dts[2] < dts[1] < dts[0]
    if captured:
        f.capture_run(ur, work, dt_r, 3, 0.05).launch()
    else:
        f.run(ur, work, dt_r, 3, 0.05)
    assert abs(_host(dt_r)[0] - dts[2]) <= 1e-13 * dts[2]
    # (the y and z momenta are zero up to rounding)
    assert rel_diff_floored(_host(ur)[-1:], _host(us)[-1:], floor=1e-2).max() <= 1e-13
