"""The size of the pair loop's work items: the rule itself on the host, and masked
passes over every particle bitwise against plain passes, at dense cells that
both cut into sub-items.  (Masked passes over some of the particles follow the
FP64 oracle in test_gpu_ml.py.)"""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <hip/hip_runtime.h>
#include "sr_internal.h"

int main()
{
    for (int b = 10; b < 45; ++b) {
        const unsigned long long work = 1ull << b;
        // a partial pass of 2^13 pairs or more makes an item per 2^13 pairs until
        // there are two items for each of 8192 wavefronts
        const unsigned long long want = work >> 13 < 16384 ? work >> 13 : 16384;
        if (want && work / item_pairs(work, true) < want) {
            std::printf("2^%d pairs: items of %lld\n", b, item_pairs(work, true));
            return 1;
        }
        if (item_pairs(work, false) < item_pairs(work, true) || item_pairs(work, false) < 65536)
            return 2;
    }
    return 0;
}
"""


def test_partial_passes_make_enough_items(tmp_path):
    src = tmp_path / "cut.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "cut"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip",
                    "--offload-host-only", "-std=c++17", "-w", "-I",
                    os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1410_2805_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout


R_MAX, EPS, CELL, L = 3.0, 0.1, 3.0, 16.0


def _dense(count, seed):
    """A cell of `count` particles in a sparse box, all kept 1e-5 away from the
    cell faces so that float32 offsets and FP64 positions agree on every cell."""
    rng = np.random.default_rng(seed)
    h = L / int(L // CELL)
    pos = np.concatenate([h * (2.0 + rng.random((count, 3))), L * rng.random((700, 3))])
    fr = pos / h - np.floor(pos / h)
    pos = np.where(fr < 1e-5, pos + 2e-5, np.where(fr > 1 - 1e-5, pos - 2e-5, pos))
    pos = np.mod(pos, L)
    vel = rng.normal(scale=0.1, size=pos.shape).astype(np.float32)
    return pos, vel, np.ones(pos.shape[0], np.float32)


def _step(pos, vel, m, n_sub, ml, dt=0.02):
    import torch

    from paper_1410_2805_amd import gridfit, sr
    ctx = sr.Context(0)
    pm = sr.PM(ctx, 16, L)
    box = sr.Box.make(L)
    dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0", t)
    c3, ox, oy, oz = sr.sr_split_from_f64(ctx, *(dev(pos[:, d], torch.float64) for d in range(3)),
                                          box, CELL)
    st = {"cell3": c3, "ox": ox, "oy": oy, "oz": oz, "m": dev(m, torch.float32)}
    for d, k in enumerate(("vx", "vy", "vz")):
        st[k] = dev(vel[:, d], torch.float32)
    lr = tuple(torch.zeros_like(st["m"]) for _ in range(3))
    so = tuple(torch.zeros_like(st["m"]) for _ in range(3))
    sr.sr_ksk_step(ctx, pm, st, box,
                   sr.StepParams.make(R_MAX, EPS, gridfit.poly_coeffs(), CELL, dt, n_sub, ml=ml),
                   lr, False, so)
    x = torch.stack(sr.sr_split_to_f64(ctx, st["cell3"], st["ox"], st["oy"], st["oz"], box, CELL),
                    1)
    v = torch.stack([st["vx"], st["vy"], st["vz"]], 1)
    ctx.sync()
    x, v = x.cpu().numpy(), v.double().cpu().numpy()
    pm.close()
    ctx.close()
    return x, v


@pytest.mark.gpu
@pytest.mark.parametrize("count", [128, 1100, 9000])
def test_full_mask_equals_plain_pass(count):
    pos, vel, m = _dense(count, count)
    a = _step(pos, vel, m, 1, (10 ** 6, 2, 2))
    b = _step(pos, vel, m, 2, None)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
