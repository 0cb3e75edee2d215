"""Rules that size a launch, compiled from the library's own header for the
host (launch_rules_check.cpp), over ranges that no GPU test could allocate."""
import os
import shutil
import subprocess

import pytest

from test_gpu_segments import CASES, LARGE

SEGMENTED = CASES + LARGE
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    cxx = shutil.which("g++")
    rocm = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    if cxx is None or not os.path.isdir(os.path.join(rocm, "hip")):
        pytest.skip("g++ or the HIP headers are missing")
    out = str(tmp_path_factory.mktemp("rules") / "check")
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-D__HIP_PLATFORM_AMD__", "-isystem", rocm,
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2606_20537_amd", "csrc"),
                    os.path.join(ROOT, "tests", "launch_rules_check.cpp"), "-o", out], check=True)
    return out


def run(exe, *args):
    return subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()


@pytest.fixture(scope="module")
def lines(exe):
    return run(exe)


@pytest.mark.parametrize("rule", ["fp8_grid", "gather_shares", "placement", "segments"])
def test_rule(lines, rule):
    assert rule + " ok" in lines, lines


@pytest.mark.parametrize("case", SEGMENTED, ids=lambda c: "%d_%d_%d_%d_%s" % c[:5])
def test_segmented_cases_have_their_plan(exe, case):
    T, H, dk, dv, dtype, states, _, plan = case
    assert run(exe, T, H, dk, dv, int(dtype == "f32"), int(states)) == [" ".join(map(str, plan))]
