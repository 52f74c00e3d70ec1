"""Batches whose pass-1 rows exceed the memory-side cache, of one segment and of
several: the same bits as through a workspace of a few points, whose launches
store the other way."""
import numpy as np
import pytest
import torch

import synth
from tests._cases import Case
from tests._gpu import dev, make_ctx, require_gpu, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("names,n,points,prec", [("HLV", 16384, 1025, 0), ("HL", 65536, 260, 0), ("HL", 16384, 520, 1)])
def test_store_policy_keeps_the_bits(names, n, points, prec):
    require_gpu()
    cases = [Case(names, n, 2048.0, snr=13.0, cfg=26, realization=r, psd="network") for r in range(2)]
    lo, hi = synth.SEARCH_BOX_30HZ_LO, synth.SEARCH_BOX_30HZ_HI
    th = torch.from_numpy(synth.uniform_in_box(np.random.default_rng(9), points, lo, hi)).to(dev())
    whole = make_ctx(cases[0], prec, max_batch=points, max_segments=2)
    few = make_ctx(cases[0], prec, max_batch=points, max_segments=2, workspace_bytes=7 * 2 * n * (16 if prec else 8))
    assert whole.workspace_bytes >= 1 << 28
    for ctx in (whole, few):
        for s in range(2):
            upload(ctx, s, cases[s])
    k = torch.arange(points, dtype=torch.int32, device=dev())
    for seg in (0 * k, k % 2, (k >= points // 2).to(torch.int32)):   # one, in turn, one after the other
        a, b = whole.eval(th, seg.contiguous()), few.eval(th, seg.contiguous())
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    whole.close()
    few.close()
