"""The FP64 thread-per-cell stage contracting one axis at a time, where its
tiles can go wrong: block sizes that leave partial waves, every slab height
(one row or layer, uneven counts of extra faces, the whole leaf), hanging
faces in both directions, outflow and periodic faces, the limiter and
mortar faces, against the oracle.  The tolerance is the parity tests' bar
(three steps of round-off on states of order one)."""
import numpy as np
import pytest

from paper_2502_12620_amd import workloads as W
from tests.gpu_helpers import make_pair, rel_diff
from tests.test_gpu_parity import TOL, _cuda, _forest, _host, _physical_state

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (dim, degree, N, slab rows): N = 2 (four-cell leaves), one-row slabs,
# odd row counts, partial last waves, the largest blocks in one workgroup
CASES = [(2, 0, 2, 0), (2, 1, 6, 1), (2, 1, 10, 5), (2, 2, 6, 3), (2, 2, 16, 16), (2, 3, 10, 2), (2, 3, 12, 12),
         (3, 0, 2, 0), (3, 1, 2, 2), (3, 1, 6, 3), (3, 1, 8, 8), (3, 1, 8, 2)]


@pytest.mark.parametrize("dim,p,N,rows", CASES)
@pytest.mark.parametrize("mode", ["plain", "limiter", "conservative"])
def test_slab_shapes_against_the_oracle(dim, p, N, rows, mode):
    from paper_2502_12620_amd import dgamr as G

    w = _forest(dim, p, N, 3 if N <= 6 else 2, bc=W.OUTFLOW if mode == "plain" else W.PERIODIC)
    orc, gpu = make_pair(w, hanging=1 if mode == "conservative" else 0, limiter=mode == "limiter")
    gpu.set_tuning(G.TUNE_STAGE_VARIANT, 1)
    gpu.set_tuning(G.TUNE_SLAB_ROWS, rows)
    u = _physical_state(orc, w, seed=11 + 10 * p + N)
    ud, work, dt = _cuda(u), gpu.new_work(), torch.zeros(1, dtype=torch.float64, device="cuda")
    gpu.run(ud, work, dt, 3, 0.1)
    for _ in range(3):
        orc.step(u, 0.1, limiter=mode == "limiter")
    got = _host(ud)
    assert np.isfinite(got).all()
    assert rel_diff(got, u).max() <= TOL


# The residual alone on the thread-per-cell kernel (the lane kernel takes small
# forests): automatic slabs at block sizes that fill whole and partial waves,
# one-row slabs; heights that are no divisor, or past the lane kernel's 512
# threads, stay refused for the 2-D residual.
@pytest.mark.parametrize("dim,p,N,rows", [(2, 0, 6, 0), (2, 1, 10, 1), (2, 1, 12, 0), (2, 2, 10, 0), (2, 2, 16, 16),
                                          (2, 3, 4, 0), (2, 3, 16, 0), (2, 3, 12, 3), (3, 1, 6, 2)])
def test_residual_alone_against_the_oracle(dim, p, N, rows):
    from paper_2502_12620_amd import dgamr as G

    w = _forest(dim, p, N, 3 if N <= 6 else 2, bc=W.OUTFLOW if rows else W.PERIODIC)
    orc, gpu = make_pair(w, hanging=0)
    gpu.set_tuning(G.TUNE_STAGE_VARIANT, 1)
    gpu.set_tuning(G.TUNE_SLAB_ROWS, rows)
    u = _physical_state(orc, w, seed=3 + p + N)
    ud, gd, rd = _cuda(u), gpu.new_guard(), gpu.new_residual()
    gpu.fill_guardcells(ud, gd)
    if dim == 2 and rows * N * 4 > 512:
        with pytest.raises(G.DgamrError):
            gpu.dg_residual(ud, gd, rd)
        return
    gpu.dg_residual(ud, gd, rd)
    assert rel_diff(_host(rd), orc.residual(u)).max() <= TOL
    with pytest.raises(G.DgamrError):  # a slab height that is no divisor
        gpu.set_tuning(G.TUNE_SLAB_ROWS, N - 1 if N > 2 else 3)
        gpu.dg_residual(ud, gd, rd)
