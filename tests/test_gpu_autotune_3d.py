"""The autotuner on a 3-D pool that takes the lane kernel by default: its
choice includes the kernel's own slab height (whole blocks from 1024 leaves on,
which no height that can be asked for gives), so that the tuned stage is no
slower than the default one (the slabs of two layers it once chose from take
a z face more for every layer: a fifth of the time).  The bar is a tenth, several
times what repeated timings of one shape differ by."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_tuned_3d_pool_is_no_slower_than_the_default():
    from paper_2502_12620_amd import dgamr as G

    roots = (16, 16, 4)
    f = G.Forest(3, 3, 8, roots, (0.0,) * 3, tuple(map(float, roots)), (0,) * 3, 1, 1.4)
    pool = G.Pool(3, 3, 8, capacity_leaves=1024, max_members=1)
    mid, first = pool.admit(f, 0.05)
    pool.u.zero_()
    pool.view(first, f.n_leaves)[:, 0, 0] = 1.0
    pool.view(first, f.n_leaves)[:, 4, 0] = 2.5

    def step_us():
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        best = 1e30
        for _ in range(4):
            e0.record()
            pool.step()
            e1.record()
            e1.synchronize()
            best = min(best, 1e3 * e0.elapsed_time(e1))
        return best

    before = step_us()
    variant, rows, grid, us = pool.autotune()
    tuned = step_us()
    pool.set_lanes(0)  # the default shape again: both sides after the same load
    default = step_us()
    print(f"default {before:.1f} / {default:.1f} us a step, tuned {tuned:.1f} (variant {variant}, rows {rows}, grid {grid}, {us:.1f} us a stage)")
    assert tuned <= 1.1 * max(before, default)
