"""The stage runtime on a simulated device, without a GPU: tests/host/stage_runtime_test.cpp compiles stage.cpp into itself and
checks the order in which it has kernels read and write, the passes it forms and the calls it accepts."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_stage_runtime_on_a_simulated_device(tmp_path):
    clang = shutil.which("clang++", path=os.path.join(ROCM, "llvm", "bin"))
    if not clang:
        pytest.skip("no clang++")
    exe = str(tmp_path / "stage_runtime")
    # every function that a simulated call replaces is defined in the program: nothing of the HIP runtime is linked
    r = subprocess.run([clang, "-std=c++17", "-O1", "-Wall", "-Wno-unused-function", "-Werror", "-D__HIP_PLATFORM_AMD__",
                        "-I" + os.path.join(ROCM, "include"), os.path.join(HERE, "host", "stage_runtime_test.cpp"),
                        "-o", exe, "-pthread"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert "all checks passed" in r.stdout
