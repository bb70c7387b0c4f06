"""A serving slot's workspace holds what every one of its graphs uses
(csrc/serve_plan.hpp, which serve.hip sizes a slot and captures its graphs
with): tests/host_serve/slot_workspace.cpp plans random matrices on the host,
under AddressSanitizer and UndefinedBehaviorSanitizer.

A graph that used more would write past the slot's device allocation, on the
launch that sets the slot up already, so this is checked on the host for every
bucket of right-hand sides and for chunked passes."""
import os
import shutil
import subprocess
import warnings

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "host_serve", "slot_workspace.cpp")
INC = os.path.join(os.path.dirname(HERE), "paper_1902_08018_amd", "csrc")


@pytest.fixture(scope="module")
def slots(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not found")
    out = str(tmp_path_factory.mktemp("slot") / "slot_workspace")
    base = [gxx, "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", INC, SRC, "-o", out]
    r = subprocess.run(base + ["-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"],
                       capture_output=True, text=True)
    if r.returncode != 0:
        warnings.warn("sanitizers unavailable: plain build")
        r = subprocess.run(base + ["-O2"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


@pytest.mark.parametrize("seed,most_rows,most_values", [(1, 65536, 2 ** 29), (2, 4000, 2 ** 26), (3, 2000000, 2 ** 31)])
def test_every_bucket_fits_the_slot(slots, seed, most_rows, most_values):
    r = subprocess.run([slots, "fit", str(seed), "20000", str(most_rows), str(most_values)], capture_output=True,
                       text=True, env={**os.environ, "ASAN_OPTIONS": "detect_leaks=0"}, timeout=120)
    assert r.returncode == 0, f"exit {r.returncode}:\n{r.stderr[-2000:]}"


# (rate, rows, columns, values a chunk): bytes, from the rules for 1 (lanes of
# the rate), 16 (16 waves) and 32, 48 and 64 (8 waves) right-hand sides: about
# two rounds of workgroups in a multiple of 8 slabs, within 256 MiB.  A slot's
# bytes decide what a budget admits, so they do not follow the planners' costs
# (which would double the first one).
SIZES = {(24, 18237, 28044, 1 << 28): 85499904, (8, 40000, 256, 1 << 28): 82018304,
         (16, 43412, 168, 1 << 28): 66754560, (8, 1024, 1024, 1 << 28): 8781824,
         (8, 65536, 65536, 1 << 28): 92274688, (32, 2048, 1024, 69632): 950272,
         (4, 8981, 58363, 1 << 28): 96010240}


@pytest.mark.parametrize("shape", list(SIZES))
def test_slot_size(slots, shape):
    r = subprocess.run([slots, "size", *map(str, shape)], capture_output=True, text=True,
                       env={**os.environ, "ASAN_OPTIONS": "detect_leaks=0"}, timeout=60)
    assert r.returncode == 0, r.stderr
    assert int(r.stdout) == SIZES[shape]
