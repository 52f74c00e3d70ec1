"""Every two-pass plan at the edges of its work split: one point and a number
of points that leaves the last group short, networks of one to eight
detectors, points outside the rectangle, two segments in turn (pass 1 keeps a
segment's data between points), and a restricted coalescence range (the general
reduction of pass 2), against the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import fitness as F
from tests._cases import Case
from tests._gpu import assert_parity, dev, make_ctx, require_gpu, upload

pytestmark = pytest.mark.gpu

NAMES = ("L", "HL", "HLV", "HLVK", "HLVKH", "HLVKHL", "HLVKHLV", "HLVKHLVK")


def _plans():
    from paper_2002_02150_amd import fcas
    try:
        return [(p, d["n"]) for p, d in fcas.plans() if d["n"] <= 262144]
    except RuntimeError:   # library not built: nothing to run on the CPU either
        return []


# parity bars of the fitness: 1e-4 relative (mixed), 1e-9 (FP64)
@pytest.mark.parametrize("prec,rtol", [(0, 1e-4), (1, 1e-9)], ids=["mixed", "fp64"])
@pytest.mark.parametrize("plan,n", _plans())
def test_plan_edges(plan, n, prec, rtol):
    require_gpu()
    names = NAMES[(plan + 3 * prec) % 8]
    fs = 1024.0 if n <= 8192 else 2048.0
    cases = [Case(names, n, fs, snr=12.0, cfg=60, realization=r, psd="network") for r in range(2)]
    lo, hi = synth.SEARCH_BOX_30HZ_LO, synth.SEARCH_BOX_30HZ_HI
    rng = np.random.default_rng(61 + plan)
    ctx = make_ctx(cases[0], prec, max_batch=9, max_segments=2)
    ctx.select_plan(plan, 1 + plan, 3 * n // 512)   # grids of less and more than a group of work-groups
    for s in range(2):
        upload(ctx, s, cases[s])
    th = synth.uniform_in_box(rng, 9, lo, hi)
    th[::2] = synth.near_point(rng, 5, cases[0].theta0, lo, hi, 0.01)
    th[3, 0] = 7.0                                   # outside
    seg = np.array([0, 1, 0, 0, 1, 1, 0, 1, 0], dtype=np.int32)
    box = (np.array(lo), np.array(hi))

    def run(rows):
        f, j = ctx.eval(torch.from_numpy(th[rows].copy()).to(dev()), torch.from_numpy(seg[rows].copy()).to(dev()))
        return f.cpu().numpy(), j.cpu().numpy()

    f, j = run(np.arange(9))
    for s in range(2):
        rows = np.nonzero(seg == s)[0]
        fo, jo = F.fitness_batch(cases[s].seg, cases[s].net.pos_m, cases[s].net.tensor, th[rows], *box)
        assert_parity(cases[s], th[rows], f[rows], j[rows], fo, jo, rtol)
    f1, j1 = run(np.array([6]))
    assert f1[0] == f[6] and j1[0] == j[6]
    lo_j, hi_j = n // 3 + 1, n // 3 + 1 + n // 7
    ctx.set_segment_range(0, lo_j, hi_j)
    f, j = run(np.nonzero(seg == 0)[0])
    for k, row in enumerate(np.nonzero(seg == 0)[0]):
        fo, jo = F.fitness(cases[0].seg, cases[0].net.pos_m, cases[0].net.tensor, th[row], *box, j_range=(lo_j, hi_j))
        if not np.isfinite(fo):
            assert f[k] == -np.inf and j[k] == -1
            continue
        assert abs(f[k] - fo) <= rtol * fo and lo_j <= j[k] < hi_j
        assert j[k] == jo or F.gamma2_at(cases[0].seg, cases[0].net.pos_m, cases[0].net.tensor, th[row],
                                         int(j[k])) >= (1 - 1e-4) * fo
    ctx.close()
