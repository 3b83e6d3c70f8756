"""The window tile of the pair loop (sr_item.h): for every number of lane groups
S, every entry that a pass writes or reads lies inside it.  A small host
program, built from the headers the kernels are built from, follows the number
of staged sources through all counts that windows can keep; the same clumps
that reach the largest counts are summed on the GPU against the FP64 oracle."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <hip/hip_runtime.h>
#include "sr_item.h"

int main()
{
    constexpr ItemTables tab = make_item_tables();
    constexpr int entries = sizeof(ItemShared::tile) / sizeof(float4);
    int bad = 0;
    for (int S = 1; S <= kMaxSplit; ++S) {
        const int q = 2 * S;
        bool seen[2 * entries] = {true};  // sources a tile may keep before a window
        int most = 0;
        for (bool more = true; more;) {
            more = false;
            for (int kept = 0; kept < entries; ++kept)
                if (seen[kept])
                    for (int add = 0; add <= kWindow; ++add) {
                        const int fill = kept + add;
                        const int n = (fill * tab.srecip[S]) >> 16;
                        if (n != fill / q)
                            ++bad;
                        // the last window: the last quantum is filled up
                        const int end = (fill + q - 1) / q * q;
                        most = end > most ? end : most;
                        // another follows: the tile keeps its sources, or a pass
                        // takes the whole quanta
                        const int next = fill <= tab.hold[S] ? fill : fill - n * q;
                        if (!seen[next])
                            more = seen[next] = true;
                    }
        }
        if (most > entries)
            std::printf("S=%d: %d entries of %d\n", S, most, entries), ++bad;
    }
    return bad != 0;
}
"""


def test_staged_sources_stay_in_the_tile(tmp_path):
    src = tmp_path / "stage.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "stage"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip",
                    "--offload-host-only", "-std=c++17", "-w", "-I",
                    os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1410_2805_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout


# Targets on one side of a cell face (3, 5, 6, 7, 9, 10 and 12 lane groups and
# two targets per lane), in a clump of `total` particles that all pass the box
# test: the last window then finds 64 sources staged and adds total - 64.
@pytest.mark.gpu
@pytest.mark.parametrize("total", [121, 122, 123, 124, 125, 126, 127, 128])
@pytest.mark.parametrize("near", [5, 6, 7, 9, 10, 12, 17, 21, 33, 41])
def test_clump_across_a_cell_face(near, total):
    from oracle import oracle as O
    from paper_1410_2805_amd import gridfit, sr
    from paper_1410_2805_amd import workloads as W
    from tests.parity import accel_np, check_accel, to_dev
    rng = np.random.default_rng(1000 * near + total)
    L = 15.0
    pos = 7.25 + 0.5 * rng.random((total, 3))
    side = np.arange(total) < near
    pos[:, 0] = np.where(side, 5.75, 6.05) + 0.2 * rng.random(total)  # the face is at 6
    p = W._soa(pos[rng.permutation(total)], L)
    p.m[:] = np.exp(0.5 * rng.standard_normal(p.n)).astype(np.float32)
    poly = gridfit.poly_coeffs()
    ctx = sr.Context(0)
    t = to_dev(p)
    a = accel_np(*sr.sr_force(ctx, t["x"], t["y"], t["z"], t["m"], sr.Box.make(L), 3.0, 3.0, 0.1,
                              poly)[:3])
    ctx.sync()
    ref = O.force(p.x, p.y, p.z, p.m, L, 3.0, 0.1, poly.astype(np.float64))
    check_accel(a, ref, "%d of %d" % (near, total))
