"""bq_step_plan_create when the host's memory runs out (tests/c/plan_alloc_failure.cpp):
an error, no plan, nothing left allocated, whichever allocation fails."""
import os
import subprocess

import pytest

from paper_2110_02861_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(os.environ.get("BQ_SANITIZE") == "1",
                    reason="the sanitizer's runtime replaces operator new itself")
def test_plan_creation_frees_everything_when_an_allocation_fails(tmp_path):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    lib = os.path.dirname(build.LIB)
    exe = str(tmp_path / "plan_alloc_failure")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(build.ROOT, "include"), "-I", os.path.join(rocm, "include"),
                    os.path.join(HERE, "c", "plan_alloc_failure.cpp"), "-o", exe, "-rdynamic",
                    "-L", lib, "-lbq", "-L", os.path.join(rocm, "lib"), "-lamdhip64",
                    f"-Wl,-rpath,{lib}", f"-Wl,-rpath,{os.path.join(rocm, 'lib')}"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "plan_alloc_failure ok" in r.stdout, r.stdout + r.stderr
