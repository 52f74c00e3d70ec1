"""Which lengths the fused schedule takes in one launch, and that a context of
it gives the two-pass results, bit for bit, on both sides of that line: fitness
batches small and large, mixed lengths, the polish and whole iterations."""
import numpy as np
import pytest
import torch

import synth
from tests._cases import Case
from tests._gpu import dev, make_ctx, require_gpu, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths,fused_launches", [((8192,), 1), ((16384,), 0), ((131072,), 0), ((4096, 24576), 1)])
def test_fused_line(lengths, fused_launches):
    require_gpu()
    from paper_2002_02150_amd import PsoConfig, Swarm, polish
    cases = [Case("HLV", n, 2048.0, snr=13.0, cfg=26, psd="network") for n in lengths]
    lo, hi = synth.SEARCH_BOX_30HZ_LO, synth.SEARCH_BOX_30HZ_HI
    out = []
    for schedule in (0, 1):
        ctx = make_ctx(cases[0], 0, max_batch=80, max_segments=2, max_samples=max(lengths), schedule=schedule)
        for s, case in enumerate(cases):
            upload(ctx, s, case)
        got = []
        for points in (1, 3, 80):
            th = np.random.default_rng(points)
            th = torch.from_numpy(synth.uniform_in_box(th, points, lo, hi)).to(dev())
            seg = (torch.arange(points, dtype=torch.int32, device=dev()) % len(lengths)).contiguous()
            ctx.set_timing(True)
            got += [t.clone() for t in ctx.eval(th, seg)]
            assert ctx.read_timing("fused")[1] == (fused_launches if schedule == 0 else 0)
            ctx.read_timing("pass1"), ctx.read_timing("pass2")
            ctx.set_timing(False)
        th = torch.from_numpy(synth.near_point(np.random.default_rng(7), 4, cases[0].theta0, lo, hi, 0.01)).to(dev())
        seg = torch.zeros(4, dtype=torch.int32, device=dev())
        got += [t.clone() for t in polish(ctx, th, seg, steps=2, trials=4)]
        sw = Swarm(ctx, PsoConfig(n_runs=2, n_particles=20, n_iter=50, seed=3))
        sw.init()
        f = torch.empty(40, dtype=torch.float64, device=dev())
        j = torch.empty(40, dtype=torch.int32, device=dev())
        sw.run(3, torch.zeros(40, dtype=torch.int32, device=dev()), f, j)
        got += [f, j, sw.theta.clone(), sw.best_f.clone()]
        assert ctx.device_error() == 0
        out.append(got)
        ctx.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)
