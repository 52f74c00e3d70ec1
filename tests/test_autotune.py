"""The calls of the autotuner."""
import inspect
import json

import pytest

from paper_2002_02150_amd import autotune as A


def test_arguments_of_earlier_calls_bind():
    b = inspect.signature(A.autotune).bind((8192,), 4, 2048.0, 256, 10, (1024, 2048), "t.json", 0, print)
    assert b.arguments["batch"] == 256 and b.arguments["grids"] == (1024, 2048) and b.arguments["out"] == "t.json"


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
