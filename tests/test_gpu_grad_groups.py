"""fitness_grad_batch over every detector group of the adjoint kernel (two to
eight detectors: one group of up to four, or two groups, the last of them
short), lengths that are and are not powers of two, and batches from one point
(split into the most parts) up, against the oracle's gradient."""
import numpy as np
import pytest
import torch

import synth
from oracle import gradient as G
from tests._cases import Case
from tests._gpu import dev, make_ctx, require_gpu, upload

pytestmark = pytest.mark.gpu


# bars of the gradient (components in rectangle-width units, s the largest):
# every component within tol s, every component above 1e-3 s within rtol of itself
@pytest.mark.parametrize("prec,tol,rtol", [(0, 1e-5, 1e-4), (1, 1e-10, 1e-9)], ids=["mixed", "fp64"])
@pytest.mark.parametrize("names,n,points", [
    ("HL", 8192, 1), ("HLV", 24576, 3), ("HLVK", 49152, 1), ("HLVKH", 8192, 5), ("HLVKHL", 24576, 2),
    ("HLVKHLV", 8192, 1), ("HLVKHLVK", 24576, 3),
])
def test_gradient_detector_groups(names, n, points, prec, tol, rtol):
    require_gpu()
    case = Case(names, n, 1024.0 if n == 8192 else 2048.0, snr=12.0, cfg=23, psd="network")
    lo, hi = synth.SEARCH_BOX_30HZ_LO, synth.SEARCH_BOX_30HZ_HI
    rng = np.random.default_rng(24)
    th = synth.near_point(rng, points, case.theta0, lo, hi, 0.01)
    ctx = make_ctx(case, prec, max_batch=points)
    upload(ctx, 0, case)
    f, j, g = ctx.grad(torch.from_numpy(th).to(dev()), torch.zeros(points, dtype=torch.int32, device=dev()))
    j, g = j.cpu().numpy(), g.cpu().numpy()
    w = np.array(hi) - np.array(lo)
    for k in range(points):
        _, _, go = G.fitness_gradient(case.seg, case.net.pos_m, case.net.tensor, th[k], int(j[k]))
        scale = np.max(np.abs(go * w))
        err = np.abs((g[k] - go) * w)
        assert np.all(err <= tol * scale), (k, g[k], go)
        big = np.abs(go * w) > 1e-3 * scale
        assert np.all(err[big] <= rtol * np.abs(go * w)[big]), (k, g[k], go)
    ctx.close()
