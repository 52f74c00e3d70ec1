"""The stages of the main passes with their twiddle factors in registers, on
the CPU: every transform shape of the plans, both precisions, against the
direct sum in extended precision."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_geo_stages_match_direct_sum(tmp_path):
    src = os.path.join(ROOT, "tests", "emu", "geo_check.cpp")
    exe = str(tmp_path / "geo_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined",
                    "-I" + os.path.join(ROOT, "paper_2002_02150_amd", "csrc"), src, "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split("\n")
    rows = [ln.rsplit(maxsplit=2) for ln in out if ln]
    assert len(rows) == 2 * 21
    for shape, prec, err in rows:
        # ten butterfly layers, each with a rounding of one unit and a factor
        # off by at most one and a half
        eps = 2.0 ** -24 if prec == "f32" else 2.0 ** -53
        assert float(err) <= 25 * eps, (shape, prec, err)
