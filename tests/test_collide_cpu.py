"""Host test of the collision's arithmetic (csrc/d3q19_mrt.hpp through
tests/collide_check.cpp): its rounding error against 64 bits and more, and the
momentum that FP32 steps keep at any relaxation rate."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if not os.path.exists(os.path.join(INCLUDE, "hip", "hip_runtime.h")):
        pytest.skip("needs the HIP headers")
    exe = str(tmp_path_factory.mktemp("collide") / "collide_check")
    subprocess.check_call(
        [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-w", "-ffp-contract=off",
         "-D__HIP_PLATFORM_AMD__", "-I", INCLUDE,
         "-I", os.path.join(ROOT, "paper_2512_23116_amd", "csrc"),
         os.path.join(ROOT, "tests", "collide_check.cpp"), "-o", exe])

    def run(what, s_m):
        r = subprocess.run([exe, what, str(s_m)], capture_output=True, text=True, timeout=300)
        print(r.stdout, r.stderr)
        return r.returncode

    return run


@pytest.mark.parametrize("s_m", [1.98, 0.7])
@pytest.mark.parametrize("what", ["single", "double"])
def test_collision_rounds_like_a_few_stores(check, what, s_m):
    assert check(what, s_m) == 0


@pytest.mark.parametrize("s_m", [0.49, 1.2, 1.98])
def test_single_precision_steps_keep_the_momentum(check, s_m):
    assert check("momentum", s_m) == 0


def test_any_reference_density(check):
    assert check("rho0", 1.98) == 0
