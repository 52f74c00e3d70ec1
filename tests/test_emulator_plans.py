"""The CPU emulator runs the kernels' own transforms: the plans and detector
counts that test_emulator.py leaves out, against the oracle, and a planted
mistake in the factors of pass 2's rows, which must show."""
import numpy as np
import pytest

from tests._cases import Case
from tests.test_emulator import PLANS, _run, emu  # noqa: F401 (fixture)


def _off(emu, tmp_path, plan, names, prec):  # noqa: F811
    n = PLANS[plan]
    case = Case(names, n, 1024.0 if n in (2048, 8192) else 2048.0, snr=12.0, cfg=50, realization=plan)
    theta = case.theta0 + np.array([0.01, -0.01, 0.02, 0.003])
    series, bg, bj = _run(emu, tmp_path, case, theta, plan, prec)
    ref = case.series(theta)
    assert series[bj] == bg
    return np.max(np.abs(series - ref)) / ref.max()


# bars of test_emulator.py: 2e-5 (mixed) and 1e-10 (FP64) of the peak
@pytest.mark.parametrize("plan,names,prec", [
    (10, "HLVKHLVK", 0), (11, "HLVKHLV", 0), (26, "HL", 0), (28, "L", 0), (3, "HLVKHLV", 1), (16, "HLV", 1), (34, "L", 1),
    (33, "HL", 1),
])
def test_plans_and_detector_counts(emu, tmp_path, plan, names, prec):  # noqa: F811
    assert _off(emu, tmp_path, plan, names, prec) <= (2e-5 if prec == 0 else 1e-10)


@pytest.mark.parametrize("plan,prec", [(0, 0), (8, 0), (2, 1)])
def test_a_wrong_row_shows(emu, tmp_path, monkeypatch, plan, prec):  # noqa: F811
    monkeypatch.setenv("FCAS_EMU_ROW", "1")
    assert _off(emu, tmp_path, plan, "HL", prec) > 1e-3
