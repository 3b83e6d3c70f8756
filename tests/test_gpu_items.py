"""Work items of every shape against the FP64 oracle: one cell of a given
population in a sparse periodic box, at the edges of the item shapes (targets
per lane, lane groups, windows of 64 sources) and of the chunk sizes (128, 64
and 32 targets with sub-items)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1410_2805_amd import gridfit
from paper_1410_2805_amd import workloads as W
from tests.parity import accel_np, check_accel, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("count", [1, 4, 16, 17, 31, 33, 43, 64, 65, 86, 128, 129, 256, 257, 641,
                                   3000, 6000, 12000])
def test_one_dense_cell(count, mixed):
    from paper_1410_2805_amd import sr
    rng = np.random.default_rng(1000 + count)
    L = 15.0
    dense = 6.0 + 3.0 * rng.random((count, 3))    # cell (2, 2, 2)
    pos = np.concatenate([dense, L * rng.random((211, 3))])
    p = W._soa(pos[rng.permutation(pos.shape[0])], L)
    if mixed:
        p.m[:] = np.exp(0.5 * rng.standard_normal(p.n)).astype(np.float32)
    poly = gridfit.poly_coeffs()
    ctx = sr.Context(0)
    t = to_dev(p)
    a = sr.sr_force(ctx, t["x"], t["y"], t["z"], t["m"], sr.Box.make(L), 3.0, 3.0, 0.1, poly)
    b = sr.sr_force(ctx, t["x"], t["y"], t["z"], t["m"], sr.Box.make(L), 3.0, 3.0, 0.1, poly)
    ctx.sync()
    a, b = accel_np(*a[:3]), accel_np(*b[:3])
    assert np.array_equal(a, b)
    tg = np.arange(p.n) if p.n < 4000 else np.sort(rng.choice(p.n, 2000, replace=False))
    ref = O.force(p.x, p.y, p.z, p.m, L, 3.0, 0.1, poly.astype(np.float64), targets=tg)
    check_accel(a[tg], ref, "cell of %d" % count)
