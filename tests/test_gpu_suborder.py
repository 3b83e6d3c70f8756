"""Cells whose target slots are put in sub-order before the pair loop, against
the FP64 oracle: at the edges of a segment (one round of 256 slots, 4096 slots, a
remainder of one), with degenerate boxes (a plane, a line, points) whose
particles share sub-cells, and bitwise equal between two passes."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1410_2805_amd import gridfit
from paper_1410_2805_amd import workloads as W
from tests.parity import accel_np, check_accel, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", ["box", "plane", "line", "points"])
@pytest.mark.parametrize("count", [129, 255, 257, 4096, 4097, 8449])
def test_sub_ordered_cell(count, shape):
    from paper_1410_2805_amd import sr
    rng = np.random.default_rng(2000 + count)
    L = 15.0
    dense = 6.0 + 3.0 * rng.random((count, 3))    # cell (2, 2, 2)
    if shape == "plane":
        dense[:, 1] = 7.25
    elif shape == "line":
        dense[:, 1:] = 7.25
    elif shape == "points":
        dense = dense[rng.integers(0, 5, count)]
    pos = np.concatenate([dense, L * rng.random((97, 3))])
    p = W._soa(pos[rng.permutation(pos.shape[0])], L)
    p.m[:] = np.exp(0.5 * rng.standard_normal(p.n)).astype(np.float32)
    poly = gridfit.poly_coeffs()
    ctx = sr.Context(0)
    t = to_dev(p)
    a = accel_np(*sr.sr_force(ctx, t["x"], t["y"], t["z"], t["m"], sr.Box.make(L), 3.0, 3.0, 0.1,
                              poly)[:3])
    b = accel_np(*sr.sr_force(ctx, t["x"], t["y"], t["z"], t["m"], sr.Box.make(L), 3.0, 3.0, 0.1,
                              poly)[:3])
    ctx.sync()
    assert np.array_equal(a, b)
    tg = np.arange(p.n) if p.n < 4000 else np.sort(rng.choice(p.n, 1500, replace=False))
    ref = O.force(p.x, p.y, p.z, p.m, L, 3.0, 0.1, poly.astype(np.float64), targets=tg)
    check_accel(a[tg], ref, "%s of %d" % (shape, count))
