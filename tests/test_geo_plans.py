"""The column and row transforms of every plan, with their factors in
registers, on the CPU against the direct sum in extended precision: the shapes
come from the library's own plan list, the rows from each plan's own length."""
import os
import subprocess

from tests.test_emulator import PLANS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_plan_matches_direct_sum(tmp_path):
    exe = str(tmp_path / "geo_plans")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined",
                    "-I" + os.path.join(ROOT, "paper_2002_02150_amd", "csrc"),
                    os.path.join(ROOT, "tests", "emu", "geo_plans.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split("\n")
    rows = [ln.split() for ln in out if ln]
    seen = {}
    for plan, prec, what, j1, err in rows:
        seen.setdefault((int(plan), prec, what), set()).add(int(j1))
        # at most ten butterfly layers, each a rounding of one unit and a factor
        # off by at most one and a half
        eps = 2.0 ** -24 if prec == "f32" else 2.0 ** -53
        assert float(err) <= 25 * eps, (plan, prec, what, j1, err)
    for plan, n in PLANS.items():
        for prec in ("f32", "f64"):
            assert seen[plan, prec, "columns"] == {0}
            # four rows of a two-pass plan (its first and last among them), one after a middle pass
            assert len(seen[plan, prec, "rows"]) == (4 if n <= 262144 else 1)
