"""Host test of the two-step kernel's work plans (csrc/lbm_tb2_plan.hpp through
tests/tb2_tiles_check.cpp), for both tile shapes that are launched."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_both_tile_shapes_cover_every_lattice(tmp_path):
    exe = str(tmp_path / "tb2_tiles_check")
    # the sanitizers apply to the host code only (the file has no kernels)
    subprocess.check_call(
        [HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-g", "-std=c++17",
         "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
         "-Xarch_host", "-fno-sanitize-recover=all",
         "-I", os.path.join(ROOT, "paper_2512_23116_amd", "csrc"),
         os.path.join(ROOT, "tests", "tb2_tiles_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(r.stdout, r.stderr)
    assert r.returncode == 0, r.stderr
    assert r.stdout.startswith("ok:")
