"""fitness_polish against its definition, step by step through the public
calls: numbers of trials below, at and above a group of eight, up to the most;
points outside the rectangle and of an unregistered segment; trials that leave
the rectangle; both precisions; a workspace that takes the trials in chunks."""
import numpy as np
import pytest
import torch

import synth
from tests._cases import Case
from tests._gpu import dev, make_ctx, require_gpu, upload

pytestmark = pytest.mark.gpu


def _steps(ctx, theta, seg, steps, frac, trials):
    """The polish by fitness and gradient calls (same arithmetic in FP64)."""
    lo, hi = np.array(ctx.box_lo), np.array(ctx.box_hi)
    w = hi - lo
    th = theta.copy()
    f, j = (t.cpu().numpy().copy() for t in ctx.eval(torch.from_numpy(th).to(dev()), torch.from_numpy(seg).to(dev())))
    for _ in range(steps):
        _, _, g = ctx.grad(torch.from_numpy(th).to(dev()), torch.from_numpy(seg).to(dev()))
        g = g.cpu().numpy()
        cand = np.empty((len(th), trials, 4))
        for e in range(len(th)):
            nrm = 0.0
            for d in range(4):
                nrm += (w[d] * g[e, d]) * (w[d] * g[e, d])
            nrm = np.sqrt(nrm)
            for t in range(trials):
                s = frac * 0.5 ** t
                cand[e, t] = th[e] + (s * w * w * g[e] / nrm if nrm > 0 else 0.0)
        fc, jc = ctx.eval(torch.from_numpy(cand.reshape(-1, 4)).to(dev()),
                          torch.from_numpy(np.repeat(seg, trials)).to(dev()))
        fc, jc = fc.cpu().numpy().reshape(-1, trials), jc.cpu().numpy().reshape(-1, trials)
        for e in range(len(th)):
            for t in range(trials):
                if fc[e, t] > f[e]:
                    f[e], j[e], th[e] = fc[e, t], jc[e, t], cand[e, t]
    return th, f, j


@pytest.mark.parametrize("prec", [0, 1], ids=["mixed", "fp64"])
@pytest.mark.parametrize("names,n,trials,frac,chunk", [
    ("HLVK", 16384, 1, 1e-3, 0), ("HL", 8192, 7, 1e-2, 0), ("HLV", 24576, 8, 1e-3, 3), ("HLVKH", 8192, 9, 0.5, 0),
    ("HLVK", 8192, 32, 1e-2, 5),
])
def test_polish_is_its_steps(names, n, trials, frac, chunk, prec):
    require_gpu()
    from paper_2002_02150_amd import polish
    case = Case(names, n, 1024.0 if n == 8192 else 2048.0, snr=13.0, cfg=26, psd="network")
    lo, hi = synth.SEARCH_BOX_30HZ_LO, synth.SEARCH_BOX_30HZ_HI
    rng = np.random.default_rng(27)
    th = synth.near_point(rng, 5, case.theta0, lo, hi, 0.02)
    th[1] = np.array(hi) - 1e-4 * (np.array(hi) - np.array(lo))   # trials may leave the rectangle
    th[2, 0] = 8.0                                                 # outside
    seg = np.array([0, 0, 0, 1, 0], dtype=np.int32)                # segment 1 is not registered
    ctx = make_ctx(case, prec, max_batch=5 * trials, max_segments=2,
                   workspace_bytes=chunk * 2 * n * (16 if prec else 8))
    upload(ctx, 0, case)
    want_th, want_f, want_j = _steps(ctx, th, seg, 3, frac, trials)
    t = torch.from_numpy(th.copy()).to(dev())
    _, f, j = polish(ctx, t, torch.from_numpy(seg).to(dev()), steps=3, step_frac=frac, trials=trials)
    t, f, j = t.cpu().numpy(), f.cpu().numpy(), j.cpu().numpy()
    assert np.isnan(f[3]) and j[3] == -2 and f[2] == -np.inf and j[2] == -1
    # the trials differ from these by the rounding of w^2 g / |w g| alone
    span = np.array(hi) - np.array(lo)
    assert np.all(np.abs(t - want_th) <= 1e-11 * span), (t, want_th)
    ok = np.isfinite(want_f)
    assert np.all(np.abs(f - want_f)[ok] <= 1e-5 * want_f[ok])
    assert np.array_equal(j, want_j)
    ctx.close()
