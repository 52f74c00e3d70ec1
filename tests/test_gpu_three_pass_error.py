"""Error of the mixed path at the three-pass lengths, against the FP64 path:
no larger than with all twiddles of passes 1 and 2 from tables (rms 1.34e-6 to
1.50e-6 of the fitness, the middle pass's recurrences most of it)."""
import numpy as np
import pytest
import torch

import synth
from tests._cases import Case
from tests._gpu import dev, make_ctx, require_gpu, upload

pytestmark = pytest.mark.gpu


def rms_error(names, n, points, realization):
    case = Case(names, n, 2048.0, snr=12.0, cfg=64, realization=realization)
    th = synth.uniform_in_box(np.random.default_rng(realization), points, synth.SEARCH_BOX_30HZ_LO,
                              synth.SEARCH_BOX_30HZ_HI)
    th = torch.from_numpy(th).to(dev())
    seg = torch.zeros(points, dtype=torch.int32, device=dev())
    f = []
    for prec in (0, 1):
        ctx = make_ctx(case, prec, max_batch=points, workspace_bytes=4 << 30)
        upload(ctx, 0, case)
        f.append(ctx.eval(th, seg)[0].cpu().numpy())
        ctx.close()
    return np.sqrt(np.mean((f[0] / f[1] - 1.0) ** 2))


@pytest.mark.parametrize("names,n,points", [("HLVK", 460800, 100), ("HL", 3686400, 20)])
def test_rms_error(names, n, points):
    require_gpu()
    assert np.mean([rms_error(names, n, points, r) for r in range(2)]) <= 1.3e-6
