"""sr_pair_stats against a count of the force pass's work items by hand: two cells
of a few thousand particles that meet at a corner, in a periodic box, whose chunks
the force pass halves to 64 or 32 targets.  The slots in sub-order, the chunks,
their targets' boxes and the sources within the cutoff of each box are formed in
numpy (float32 where the kernels use it)."""
import numpy as np
import pytest

from paper_1410_2805_amd import workloads as W
from tests.parity import to_dev

pytestmark = pytest.mark.gpu

SEG, MOST = 4096, 8  # slots per sub-ordered segment, sub-items per chunk at most
F = np.float32


def _sub_order(pos):
    out = []
    for s in range(0, len(pos), SEG):
        p = pos[s:s + SEG]
        lo, hi = p.min(0), p.max(0)
        inv = F(8.0) / (hi - lo)
        c = np.minimum(np.maximum((p - lo) * inv, F(0)), F(7)).astype(np.int64)
        key = np.zeros(len(p), np.int64)
        for d in range(3):
            for b in range(3):
                key |= ((c[:, d] >> b) & 1) << (3 * b + d)
        out.append(p[np.argsort(key, kind="stable")])
    return np.concatenate(out)


def _chunk_size(n):
    """Targets per full chunk of two cells of n / 2 particles whose sources are
    all n."""
    t = min(max(n * n // 2 >> 14, 1 << 16), 1 << 18)
    f = 128
    while f > 32 and n * f > MOST * t:
        f //= 2
    return f


def _kept(pos, tg):
    lo, hi = tg.min(0), tg.max(0)
    g = np.maximum(F(0), np.maximum(lo - pos, pos - hi)).astype(np.float64)
    s = (g[:, 2] * g[:, 2]).astype(F).astype(np.float64)
    s = (g[:, 1] * g[:, 1] + s).astype(F).astype(np.float64)
    s = (g[:, 0] * g[:, 0] + s).astype(F)
    return int((s < F(9.0)).sum())


def _count(pos, cells, full):
    """(least, most): full chunks exactly; a cell's last full + 1 .. 2 full targets,
    whose parts are not followed here, as one box at most, one per target at least."""
    least = most = 0
    for c in cells:
        nf = (len(c) - full - 1) // full
        for k in range(nf):
            chunk = c[k * full:(k + 1) * full]
            least += full * _kept(pos, chunk)
        rest = c[nf * full:]
        most += len(rest) * _kept(pos, rest)
        least += sum(_kept(pos, rest[k:k + 1]) for k in range(len(rest)))
        most += sum(full * _kept(pos, c[k * full:(k + 1) * full]) for k in range(nf))
    return least, most


@pytest.mark.parametrize("n,full", [(3000, 128), (4096, 128), (6018, 64), (8192, 64), (12002, 32)])
def test_candidates_are_the_force_pass_s(n, full):
    from paper_1410_2805_amd import sr
    assert _chunk_size(n) == full
    rng = np.random.default_rng(n)
    L = 15.0
    pos = 6.0 + 3.0 * rng.random((n, 3))  # cells (2, 2, 2) and (3, 3, 3) of 5 x 5 x 5
    far = rng.permutation(np.arange(n) % 2 == 1)
    p = W._soa(pos + 3.0 * far[:, None], L)
    pos = np.stack([p.x, p.y, p.z], 1)
    far = pos[:, 0] >= 9
    assert 2 * far.sum() == n and (pos[far] >= 9).all() and (pos[~far] < 9).all()
    ctx = sr.Context(0)
    t = to_dev(p)
    useful, cand, _ = sr.sr_pair_stats(ctx, t["x"], t["y"], t["z"], sr.Box.make(L), 3.0, 3.0)
    ctx.close()
    cells = [_sub_order(pos[far]), _sub_order(pos[~far])]
    least, most = _count(pos, cells, full)
    print("n=%d: candidates %d, by hand %d..%d, useful %d" % (n, cand, least, most, useful))
    assert least <= cand <= most
    # chunks of 128 targets have larger boxes: their count lies outside
    assert full == 128 or _count(pos, cells, 128)[0] > most
