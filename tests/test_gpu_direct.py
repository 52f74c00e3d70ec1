"""Small calls, whose pass 1 sets its points up itself, against the same points
through the work lists (a second length in use takes a context there): equal
bits, counts and error flags, with one point, at and beyond the most points the
direct way takes, points outside the rectangle, bad and unregistered segments,
several segments, a workspace that splits the batch, and graph replays."""
import numpy as np
import pytest
import torch

import synth
from tests._cases import Case
from tests._gpu import dev, make_ctx, require_gpu, upload

pytestmark = pytest.mark.gpu


def _points(case, n, seed):
    lo, hi = synth.SEARCH_BOX_30HZ_LO, synth.SEARCH_BOX_30HZ_HI
    rng = np.random.default_rng(seed)
    th = synth.uniform_in_box(rng, n, lo, hi)
    th[::2] = synth.near_point(rng, len(th[::2]), case.theta0, lo, hi, 0.01)
    seg = (np.arange(n) % 2).astype(np.int32)
    for k, bad in enumerate(([7.0, 0.1, 40.0, 1.2], [np.nan, 0.1, 40.0, 1.2])):
        if n > 4 + k:
            th[3 + k] = bad
    for k, s in enumerate((3, -1, 4)):   # unregistered, below and above the table
        if n > 8 + k:
            seg[7 + k] = s
    return torch.from_numpy(th).to(dev()), torch.from_numpy(seg).to(dev())


@pytest.mark.parametrize("prec", [0, 1], ids=["mixed", "fp64"])
@pytest.mark.parametrize("names,n", [("HL", 2048), ("HLVK", 8192), ("HLV", 24576), ("HLVKH", 16384),
                                     ("HLVKHLVK", 8192)])
def test_direct_equals_lists(names, n, prec):
    require_gpu()
    case = Case(names, n, 1024.0 if n <= 8192 else 2048.0, snr=13.0, cfg=26, psd="network")
    other = Case(names, 4096, case.fs, snr=13.0, cfg=26, psd="network")
    ctxs = []
    for second in (False, True):
        ctx = make_ctx(case, prec, max_batch=600, max_segments=4, max_samples=max(n, 4096))
        upload(ctx, 0, case)
        upload(ctx, 1, case)
        ctx.set_segment_range(1, n // 8, n // 2)
        if second:
            upload(ctx, 2, other)
        ctxs.append(ctx)
    split = make_ctx(case, prec, max_batch=600, max_segments=4, workspace_bytes=3 * 2 * n * (16 if prec else 8))
    upload(split, 0, case)
    upload(split, 1, case)
    split.set_segment_range(1, n // 8, n // 2)
    for points in (1, 2, 5, 16, 64, 65, 128, 129, 512, 600):
        th, seg = _points(case, points, points)
        got = []
        for ctx in (*ctxs, split):
            before = ctx.evaluated()
            f, j = ctx.eval(th, seg)
            got.append((f.cpu().numpy(), j.cpu().numpy(), ctx.evaluated() - before, ctx.device_error()))
        for other_way in got[1:]:
            assert np.array_equal(got[0][0], other_way[0], equal_nan=True), points
            assert np.array_equal(got[0][1], other_way[1]), points
            assert got[0][2:] == other_way[2:], points
        assert got[0][3] == (1 if points > 8 else 0)
    th, seg = _points(case, 6, 1)
    direct, lists = ([t.cpu().numpy() for t in c.grad(th, seg)] for c in ctxs)
    for a, b in zip(direct, lists):
        assert np.array_equal(a, b, equal_nan=True)
    for ctx in (*ctxs, split):
        ctx.close()


def test_direct_in_a_graph():
    require_gpu()
    case = Case("HLVK", 16384, 2048.0, snr=13.0, cfg=26, psd="network")
    ctx = make_ctx(case, 0, max_batch=64, max_segments=4)
    upload(ctx, 0, case)
    upload(ctx, 1, case)
    th, seg = _points(case, 7, 3)
    f, j = ctx.eval(th, seg)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.eval(th, seg, f, j)
    for k in range(4):
        new, _ = _points(case, 7, 10 + k)
        want_f, want_j = (t.clone() for t in ctx.eval(new, seg))
        th.copy_(new)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(f, want_f) and torch.equal(j, want_j)
    # a graph keeps to the length it was recorded for: a segment of another is refused
    ctx.device_error()
    upload(ctx, 1, Case("HLVK", 8192, 2048.0, snr=13.0, cfg=26, psd="network"))
    g.replay()
    torch.cuda.synchronize()
    on_0 = seg.cpu().numpy() == 0
    assert np.array_equal(f.cpu().numpy()[on_0], want_f.cpu().numpy()[on_0])
    assert torch.isnan(f)[~torch.from_numpy(on_0).to(dev())].all() and ctx.device_error() == 1
    ctx.close()
