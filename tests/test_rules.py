"""The choices the library makes from the sizes of a call, at both sides of
each line, on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "rules_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2002_02150_amd", "csrc"),
                    os.path.join(ROOT, "tests", "emu", "rules_check.cpp"), "-o", exe], check=True)

    def ask(*args):
        return int(subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True).stdout)
    return ask


def _rows(points, n, fp64=False):
    return points * 2 * n * (16 if fp64 else 8)


@pytest.mark.parametrize("nbytes,policy", [
    (_rows(109, 131072), 0), ((1 << 28) - 1, 0),      # through the L2: pass 2 finds the rows in the caches
    (1 << 28, 2), (_rows(320, 131072), 2),            # non-temporal if the launch holds several segments
    (_rows(190, 262144), 2), (_rows(100, 131072, True), 2), (1 << 30, 2),
    ((1 << 30) + 1, 1), (_rows(2048, 131072), 1),     # non-temporal
])
def test_store_policy(rule, nbytes, policy):
    assert rule("store", nbytes) == policy


@pytest.mark.parametrize("points,tiles,threads,fp64,n_det,direct", [
    (1, 32, 256, 0, 4, 1), (32, 32, 256, 0, 4, 1), (33, 32, 256, 0, 4, 0),      # 131072 float: four groups a CU
    (8, 64, 512, 0, 4, 1), (9, 64, 512, 0, 4, 0), (9, 64, 512, 0, 1, 0),        # 262144 float: two of 512 threads
    (2, 128, 1024, 0, 4, 1), (3, 128, 1024, 0, 4, 0),                           # one of 1024 threads
    (12, 64, 256, 1, 3, 1), (13, 64, 256, 1, 3, 0), (13, 64, 256, 1, 8, 0),     # 131072 double: three,
    (16, 64, 256, 1, 2, 1), (17, 64, 256, 1, 2, 0), (16, 64, 256, 1, 1, 1),     # four with up to two detectors
    (16, 64, 128, 1, 4, 1), (17, 64, 128, 1, 4, 0),                             # 98304 double: never more than four
    (448, 1, 256, 0, 4, 1), (449, 1, 256, 0, 4, 0), (448, 2, 256, 0, 6, 1),     # 2048 and 4096: points
    (448, 1, 256, 1, 2, 1), (449, 1, 256, 1, 2, 0),
    (1 << 24, 256, 512, 0, 4, 0),
])
def test_direct_calls(rule, points, tiles, threads, fp64, n_det, direct):
    """A call sets its points up in pass 1 while its work-groups start together."""
    assert rule("direct", points, tiles, threads, fp64, n_det, 256) == direct


@pytest.mark.parametrize("items,fused", [(2, 1), (8, 1), (9, 0), (16, 0), (96, 0)])
def test_fused_schedule(rule, items, fused):
    """The fused schedule takes points of few work items."""
    assert rule("fused", items) == fused


@pytest.mark.parametrize("items,grid2,fp64,groups", [
    (1024, 16384, 0, 1024), (4096, 16384, 0, 4096), (4097, 16384, 0, 4096), (4097, 2048, 0, 2048), (1 << 33, 4096, 0, 4096),
    (4097, 16384, 1, 4097), (1 << 20, 16384, 1, 16384), (1 << 33, 1, 1, 1),
])
def test_middle_pass_groups(rule, items, grid2, fp64, groups):
    assert rule("middle", items, grid2, fp64) == groups


@pytest.mark.parametrize("points,groups,bins,parts", [
    (1, 1, 62080, 64), (1, 2, 62080, 64), (16, 1, 62080, 64), (17, 1, 62080, 61), (1024, 1, 62080, 1), (1 << 24, 2, 62080, 1),
    (1, 1, 1746000, 106), (1, 1, 3492000, 213), (1, 2, 1 << 28, 256), (4, 1, 1 << 28, 256), (5, 1, 1 << 28, 205),
    (1, 1, 1, 64),
])
def test_adjoint_parts(rule, points, groups, bins, parts):
    """And no more sums than a context holds: points + 1024 per detector."""
    assert rule("adjoint", points, groups, bins) == parts
    assert points * parts <= points + 1024
