"""The fused GEMV's planner with launch-shape overrides (WH_GEMV_LANES,
WH_GEMV_ROWS, WH_GEMV_SLABS), run on the host: tests/host_serve/gemv_plan.cpp.

  capture   a call is kept out of graph capture where the overridden shape
            splits the columns: forced to one slab it uses no workspace
  rows      block rows per group are taken where the workgroup's LDS holds
            their sums, and else left at one (a plan with more is no launch)
  slabs     without overrides: the slab counts that were the faster ones where
            the planner's cost and its fixed rule differ (us of either)
"""
import math
import os
import random
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "host_serve", "gemv_plan.cpp")
INC = os.path.join(os.path.dirname(HERE), "paper_1902_08018_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not found")
    out = str(tmp_path_factory.mktemp("plan") / "gemv_plan")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", INC,
                        SRC, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(rate, rows, cols, lanes=0, rpg=0, slabs=0):
        r = subprocess.run([out, *map(str, (rate, rows, cols, lanes, rpg, slabs))], capture_output=True, text=True)
        assert r.returncode == 0
        return dict(zip(("lanes", "rpg", "nslab", "slab_bc", "uncapturable"), map(int, r.stdout.split())))

    return run


@pytest.mark.parametrize("rate", [8, 16, 24, 32])
@pytest.mark.parametrize("rows,cols", [(512, 8192), (256, 1024), (4096, 4096), (61, 100)])
def test_capture_follows_the_forced_slabs(plan, rate, rows, cols):
    assert plan(rate, rows, cols, slabs=1)["uncapturable"] == 0
    for lanes in (4, 32, 256):
        p = plan(rate, rows, cols, lanes=lanes)
        assert p["uncapturable"] == (p["nslab"] > 1), (lanes, p)
        assert plan(rate, rows, cols, lanes=lanes, slabs=1)["uncapturable"] == 0
    p = plan(rate, rows, cols, slabs=3)
    assert p["uncapturable"] == (p["nslab"] > 1)


def refused_under_capture(rows, cols, rate):
    """The rule that include/wh.h states at wh_gemv."""
    R, C = -(-rows // 4), -(-cols // 4)
    L, most = (1024, 512) if rate <= 16 else (768, 256)
    G = 8 if C >= 8 else 4
    while G < most and 10 * R < 9 * -(-R // (L // G)) * (L // G):
        G *= 2
    n = min(16, max(3, (R * C + 1024 * L) // (2048 * L)))
    if R * C > 2 ** 27:
        n = min(48, R * C // (8192 * L))
    return C > G * n


def test_capture_rule_of_the_header(plan):
    rng = random.Random(5)
    for _ in range(300):
        rows = round(math.exp(rng.uniform(0, math.log(3e6))))
        cols = max(1, round(math.exp(rng.uniform(0, math.log(min(3e5, 2e10 / rows))))))
        rate = rng.choice((2, 4, 6, 8, 10, 12, 14, 16, 20, 24, 32))
        p = plan(rate, rows, cols)
        assert p["uncapturable"] == refused_under_capture(rows, cols, rate), (rows, cols, rate)
        assert p["uncapturable"] or p["nslab"] == 1


def test_capture_without_overrides(plan):
    # one slab by cost, but several by the rule that decides: refused as before
    p = plan(16, 256, 1024)
    assert p["nslab"] == 1 and p["uncapturable"] == 1
    p = plan(8, 61, 100)  # 25 block columns: one slab by the rule too
    assert p["nslab"] == 1 and p["uncapturable"] == 0


@pytest.mark.parametrize("rate", [2, 4, 6, 8, 10, 12, 14, 16, 20, 24, 32])
@pytest.mark.parametrize("rpg", [2, 4])
def test_rows_per_group(plan, rate, rpg):
    # the rates whose staged blocks and tables leave room for the sums in half a CU's LDS
    taken = rpg if rate <= 12 or rate == 20 else 1
    assert plan(rate, 4096, 4096, lanes=64, rpg=rpg)["rpg"] == taken


@pytest.mark.parametrize("rate,rows,cols,nslab", [
    (4, 241, 45201, 236),    # 22.4; 28.4 with 707 slabs
    (6, 188, 54946, 72),     # 20.5; 25.1 with 215
    (16, 52783, 627, 7),     # 44.9; 52.6 with 5
    (32, 10209, 1848, 20),   # 56.7; 66.7 with 15
    (16, 4096, 4096, 64),    # 32.1; 38.7 with the rule's 43
    (8, 10000, 10000, 63),   # 101.5; 108.5 with the rule's 105
    (32, 26, 135831, 67),    # 26.8; 32.5 with the rule's 23
    (20, 16384, 16384, 64),  # B^T u of 64 block columns fits LDS: 301; 319 with 57 slabs of 72
    (24, 16384, 16384, 64),  # 316; 342
    (32, 16384, 16384, 64),  # 427; 445 with 32 of 128
])
def test_slabs_of_cost_and_rule(plan, rate, rows, cols, nslab):
    assert plan(rate, rows, cols)["nslab"] == nslab
