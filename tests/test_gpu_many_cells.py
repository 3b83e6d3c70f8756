"""Meshes at the edges of the work list's cell counts (one or four cells per
thread of the gather beyond 2^17 cells, 256 or 1024 cells per block of items from
2^18 on), mostly empty, against the FP64 oracle; and a batch beyond 2^17 cells
whose boxes share threads and blocks, one of them with a pair total that decides
its cut, bitwise against each box alone."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1410_2805_amd import gridfit
from paper_1410_2805_amd import workloads as W
from tests.parity import accel_np, check_accel, to_dev

pytestmark = pytest.mark.gpu

R_MAX, EPS, CELL = 3.0, 0.1, 3.0


def _clumps(nc, counts, rng):
    """Clumps of the given counts in cells spread over the mesh, the first one in its
    last cell and the second one across the faces from it."""
    cells = [np.full(3, nc - 1), np.zeros(3)]
    cells += [2 + rng.integers(0, nc - 4, 3) for _ in counts[2:]]
    pos = np.concatenate([c + rng.random((k, 3)) for c, k in zip(cells, counts)])
    return W._soa(CELL * pos[rng.permutation(len(pos))], nc * CELL)


@pytest.mark.parametrize("nc", [50, 51, 63, 64])  # 125000, 132651, 250047, 262144 cells
def test_sparse_mesh(nc):
    from paper_1410_2805_amd import sr
    p = _clumps(nc, [300, 150, 129, 64, 513], np.random.default_rng(nc))
    poly = gridfit.poly_coeffs()
    ctx = sr.Context(0)
    t = to_dev(p)
    a = accel_np(*sr.sr_force(ctx, t["x"], t["y"], t["z"], t["m"], sr.Box.make(p.L), CELL, R_MAX,
                              EPS, poly)[:3])
    ctx.sync()
    ctx.close()
    check_accel(a, O.force(p.x, p.y, p.z, p.m, p.L, R_MAX, EPS, poly.astype(np.float64)),
                "%d^3 cells" % nc)


def test_batch_beyond_2_17_cells():
    from paper_1410_2805_amd import sr
    rng = np.random.default_rng(17)
    poly = gridfit.poly_coeffs()
    ctx = sr.Context(0)
    boxes, alone = [], []
    # boxes of 125 and 343 cells put their neighbours' cells out of step with the
    # threads' fours; 40000 particles in a cell: 1.6e9 pairs, cut by the box's total
    for nc, counts in ((5, [200, 150]), (5, [40000, 100]), (51, [300, 150, 513]), (7, [140, 90]),
                       (5, [3000, 150])):
        p = _clumps(nc, counts, rng)
        t = to_dev(p)
        box = sr.Box.make(p.L)
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
