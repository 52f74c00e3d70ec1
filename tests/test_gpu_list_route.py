"""Every two-pass plan through the work lists, against the direct calls of the
same points: equal bits.  A context takes the lists where a second length is
registered.  Consecutive points of a work-group are of different segments, of
one segment, and of segments that change now and then (pass 1 keeps a segment's
data from point to point); the grids leave the last group short, and give a
work-group one point and many."""
import numpy as np
import pytest
import torch

import synth
from tests._cases import Case
from tests._gpu import dev, make_ctx, require_gpu, upload

pytestmark = pytest.mark.gpu

NAMES = ("L", "HL", "HLV", "HLVK", "HLVKH", "HLVKHL", "HLVKHLV", "HLVKHLVK")
POINTS = 11


def _plans():
    from paper_2002_02150_amd import fcas
    try:
        return [(p, d["n"], d["n2"] // d["cols"]) for p, d in fcas.plans() if d["n"] <= 262144]
    except RuntimeError:   # library not built: nothing to run on the CPU either
        return []


@pytest.mark.parametrize("prec", [0, 1], ids=["mixed", "fp64"])
@pytest.mark.parametrize("plan,n,tiles1", _plans())
def test_list_route_equals_direct(plan, n, tiles1, prec):
    require_gpu()
    names, second = NAMES[(plan + 5 * prec) % 8], 2048 if n != 2048 else 4096
    case = Case(names, n, 1024.0 if n <= 8192 else 2048.0, snr=12.0, cfg=62, psd="network")
    other = Case(names, second, case.fs, snr=12.0, cfg=62, psd="network")
    ctxs = []
    for lists in (False, True):
        ctx = make_ctx(case, prec, max_batch=POINTS, max_segments=4, max_samples=max(n, second))
        ctx.select_plan(plan)
        for s in range(3):
            upload(ctx, s, case)
        ctx.set_segment_range(1, n // 5, n // 2)
        ctx.set_segment_range(2, 3 * n // 4, n)
        if lists:
            upload(ctx, 3, other)
        ctxs.append(ctx)
    direct, lists = ctxs
    lo, hi = synth.SEARCH_BOX_30HZ_LO, synth.SEARCH_BOX_30HZ_HI
    rng = np.random.default_rng(63 + plan)
    th = synth.uniform_in_box(rng, POINTS, lo, hi)
    th[::2] = synth.near_point(rng, len(th[::2]), case.theta0, lo, hi, 0.01)
    th[4, 0] = 7.0                                   # outside
    th = torch.from_numpy(th).to(dev())
    lists.set_timing(True)
    k = np.arange(POINTS)
    for seg in (k % 3, 0 * k, k // 4, (k * k) % 3):
        sg = torch.from_numpy(seg.astype(np.int32)).to(dev())
        # the direct context, a point a call: its pass 1 has no second point and no list
        want = [torch.cat(t) for t in zip(*([o.clone() for o in direct.eval(th[e:e + 1].contiguous(),
                                                                            sg[e:e + 1].contiguous())]
                                            for e in range(POINTS)))]
        for g1 in (1, 3 * tiles1 + 1, 1 << 20):      # a group of work-groups, three, one for each point
            lists.select_plan(plan, g1, 5 * n // 512)
            f, j = lists.eval(th, sg)
            assert torch.equal(f, want[0]) and torch.equal(j, want[1]), (seg, g1)
    # one pass-1 launch for either length in each of the twelve calls
    assert lists.read_timing("pass1")[1] == 24
    assert torch.isinf(want[0][4]) and bool(torch.isfinite(want[0][[0, 1, 2, 3, 5]]).all())
    direct.close()
    lists.close()
