"""The twiddle factors that passes 1 and 2 keep in registers, on the CPU: each
as exact as a sine and cosine of its own, in both precisions."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_factors_are_as_exact_as_a_sine_of_their_own(tmp_path):
    exe = str(tmp_path / "geo_factors")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined",
                    "-I" + os.path.join(ROOT, "paper_2002_02150_amd", "csrc"),
                    os.path.join(ROOT, "tests", "emu", "geo_factors.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split("\n")
    rows = [ln.split() for ln in out if ln]
    assert len(rows) == 2 * 5
    for radix, prec, err in rows:
        # In units u, half the type's spacing at one.  Double: the fraction of a
        # turn, at most 1/8, is rounded once (0.4 u of angle), its sine or cosine
        # series within 0.4 u, the result once (0.5 u).  Float: the fraction, at
        # most 2/3, is rounded twice (4 u of angle), a seven-term sine (3 u), the
        # result, and a product with sqrt(1/2) for one factor of radix 8 (2 u).
        assert float(err) <= (1.3 if prec == "f64" else 9.8), (radix, prec, err)
