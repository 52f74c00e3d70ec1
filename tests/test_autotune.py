"""The autotuner: how it ranks what it timed (CPU), and its calls (GPU)."""
import inspect
import json

import pytest

from paper_2002_02150_amd import autotune as A


def test_arguments_of_earlier_calls_bind():
    b = inspect.signature(A.autotune).bind((8192,), 4, 2048.0, 256, 10, (1024, 2048), "t.json", 0, print)
    assert b.arguments["batch"] == 256 and b.arguments["grids"] == (1024, 2048) and b.arguments["out"] == "t.json"


def test_unused_grid_does_not_rank():
    """16 points of 32 tiles are 512 work-groups whatever grid1: differences
    between such calls are noise and must not choose a grid1."""
    plans = [(5, dict(n2=512, cols=16)), (7, dict(n2=1024, cols=8))]   # 32 and 128 tiles
    seen = []

    def time(plan, g1, g2, m):
        seen.append((plan, g1, g2, m))
        noise = {512: 0.5, 1024: 1.0, 2048: 1.0}[g1] if m == 16 and plan == 5 else 1.0
        return noise * (1.0 if plan == 5 else 1.5) * (0.9 if m == 256 and g1 == 1024 else 1.0)

    best, results = A.rank(plans, (512, 1024, 2048), (2048, 4096), (16, 256), time)
    assert best["plan"] == 5 and best["grid1"] == 1024
    assert len(results) == 12 and len(set(seen)) == len(seen)
    assert len([c for c in seen if c[0] == 5 and c[3] == 16]) == 2     # one per grid2
    assert len([c for c in seen if c[0] == 7 and c[3] == 16]) == 6     # 2048 work-groups: grid1 counts
    best, results = A.rank([(0, dict(n2=64, cols=64))], (512, 1024), (2048,), (16, 256), lambda *a: 1.0)
    assert len(results) == 1 and best["grid1"] == 1024                 # no batch uses it: the most work-groups


@pytest.mark.gpu
def test_autotune_runs(tmp_path):
    from tests._gpu import require_gpu
    require_gpu()
    out = str(tmp_path / "t.json")
    doc = A.autotune(lengths=(2048, 8192), n_det=2, batch=32, reps=1, grids=(1024,), out=out, log=lambda s: None)
    with open(out) as fh:
        assert json.load(fh)["choices"] == doc["choices"]
    assert sorted(doc["choices"]) == ["2048", "8192"]
    assert {m["plan"] for m in doc["measurements"]} == {0, 2, 19}
