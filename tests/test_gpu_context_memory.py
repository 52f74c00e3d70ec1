"""Device memory that a context takes for each point of max_batch, and the
polish at the edge of what its descriptors hold."""
import numpy as np
import pytest
import torch

import synth
from tests._cases import Case
from tests._gpu import dev, make_ctx, require_gpu, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", [0, 1], ids=["fused", "two-pass"])
def test_bytes_per_point(schedule):
    """At 2048 samples and one detector: descriptor 624, two sets of work lists
    296, partials 8, adjoint sums 96, trials 32, and half a descriptor for the
    points of a polish (312; 32 more for the fused schedule's counters); before
    a polish kept descriptors of its own a context took 1424."""
    require_gpu()
    case = Case("L", 2048, 1024.0, snr=12.0)
    make_ctx(case, 0, max_batch=64, schedule=schedule).close()
    points = 1 << 21
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx = make_ctx(case, 0, max_batch=points, workspace_bytes=2 * 2048 * 8, schedule=schedule)
    taken = before - torch.cuda.mem_get_info()[0]
    ctx.close()
    assert taken <= 1424 * points


@pytest.mark.parametrize("prec,schedule", [(0, 1), (1, 1), (0, 0)], ids=["mixed", "fp64", "fused"])
@pytest.mark.parametrize("points", [1, 2, 7, 12])
def test_polish_of_one_trial_fills_max_batch(points, prec, schedule):
    """max_batch points with one trial each take two rounds of descriptors: the
    same result as with room for all (FP64 gradients, split alike)."""
    require_gpu()
    from paper_2002_02150_amd import polish
    case = Case("HLV", 8192, 1024.0, snr=13.0, cfg=26, psd="network")
    lo, hi = synth.SEARCH_BOX_30HZ_LO, synth.SEARCH_BOX_30HZ_HI
    start = synth.near_point(np.random.default_rng(3), points, case.theta0, lo, hi, 0.01)
    out = []
    for room in (points, 2 * points + 1):
        ctx = make_ctx(case, prec, max_batch=room, schedule=schedule)
        upload(ctx, 0, case)
        th = torch.from_numpy(start.copy()).to(dev())
        f, j = polish(ctx, th, torch.zeros(points, dtype=torch.int32, device=dev()), steps=4, step_frac=1e-3, trials=1)[1:]
        out.append((th.cpu().numpy(), f.cpu().numpy(), j.cpu().numpy(), ctx.device_error()))
        ctx.close()
    assert np.all(np.abs(out[0][0] - out[1][0]) <= 1e-11 * (np.array(hi) - np.array(lo)))
    assert np.allclose(out[0][1], out[1][1], rtol=1e-6 if prec == 0 else 1e-9, atol=0)
    assert np.array_equal(out[0][2], out[1][2]) and out[0][3] == out[1][3] == 0
