"""Sub-ordered cells in every form of the pass, against the FP64 oracle: at the
edge of a round of 512 slots, inside the box and in its last cell (whose stencil
wraps: image-shifted windows in global coordinates), in global and split
coordinates, in an open box, by persistent workgroups, and in a mesh of 35937
cells (work items of 256 cells per block)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1410_2805_amd import gridfit
from paper_1410_2805_amd import workloads as W
from tests.parity import accel_np, check_accel, check_accel_slack, position_slack, to_dev

pytestmark = pytest.mark.gpu

R_MAX, EPS, CELL = 3.0, 0.1, 3.0


def _clumps(count, nc, corner, rng):
    """A cell of `count` particles and its diagonal neighbour (across the faces for
    the last cell) of 150, in units of the cell."""
    c = nc - 1 if corner else 2
    near = np.concatenate([c + rng.random((count, 3)), (c + 1) % nc + rng.random((150, 3))])
    return CELL * near[rng.permutation(count + 150)]


@pytest.mark.parametrize("corner", [False, True])
@pytest.mark.parametrize("count", [511, 512, 513, 4608])
@pytest.mark.parametrize("form", ["global", "split", "open", "many"])
def test_sub_ordered_cell(form, count, corner):
    from paper_1410_2805_amd import sr
    rng = np.random.default_rng(3000 + count + corner)
    nc = 33 if form == "many" else 5
    L = nc * CELL
    p = W._soa(_clumps(count, nc, corner, rng), L)
    p.m[:] = np.exp(0.5 * rng.standard_normal(p.n)).astype(np.float32)
    poly = gridfit.poly_coeffs()
    box = sr.Box.make(L, periodic=form != "open")
    ctx = sr.Context(0)
    t = to_dev(p)
    if form == "split":
        c3, ox, oy, oz = sr.sr_split_from_f64(ctx, *(t[k].double() for k in "xyz"), box, CELL)

    def run(persistent):
        ctx.set_tuning(xsplit=1, order=1, persistent=persistent)
        if form == "split":
            r = sr.sr_force_split(ctx, c3, ox, oy, oz, t["m"], box, CELL, R_MAX, EPS, poly)
        else:
            r = sr.sr_force(ctx, t["x"], t["y"], t["z"], t["m"], box, CELL, R_MAX, EPS, poly)
        ctx.sync()
        return accel_np(*r[:3])

    a = run(0)
    assert np.array_equal(a, run(1))
    ctx.close()
    ref = O.force(p.x, p.y, p.z, p.m, L, R_MAX, EPS, poly.astype(np.float64),
                  periodic=form != "open")
    label = "%s cell of %d" % (form, count)
    if form == "split":
        check_accel_slack(a, ref, position_slack(ref["npair"], float(p.m.max()), CELL, EPS), label)
    else:
        check_accel(a, ref, label)


@pytest.mark.parametrize("count", [511, 512, 513, 4608])
def test_batch_of_sub_ordered_cells(count):
    """Each box of a plan bitwise as by itself."""
    from paper_1410_2805_amd import sr
    rng = np.random.default_rng(4000 + count)
    poly = gridfit.poly_coeffs()
    ctx = sr.Context(0)
    boxes, alone = [], []
    for corner in (False, True):
        p = W._soa(_clumps(count, 5, corner, rng), 15.0)
        t = to_dev(p)
        box = sr.Box.make(15.0)
        alone.append(accel_np(*sr.sr_force(ctx, t["x"], t["y"], t["z"], t["m"], box, CELL, R_MAX,
                                           EPS, poly)[:3]))
        t.update({k: torch.empty_like(t["m"]) for k in ("ax", "ay", "az")})
        t.update(box=box, cell=CELL)
        boxes.append(t)
    plan = sr.Plan(ctx, boxes, R_MAX, EPS, poly)
    plan.set_tuning(xsplit=1, order=1, persistent=0)
    plan.run()
    ctx.sync()
    for t, a in zip(boxes, alone):
        assert np.array_equal(accel_np(t["ax"], t["ay"], t["az"]), a)
    plan.close()
    ctx.close()
