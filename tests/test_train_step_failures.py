"""A training step that fails at any of its launches leaves Adam's step count
as it was (CPU: the entry point's own code over stand-ins for the launchers)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_step_count_after_a_failed_launch(tmp_path):
    cxx = shutil.which("amdclang++") or os.path.join(ROCM, "bin", "amdclang++")
    if not os.path.exists(cxx):
        pytest.skip("no amdclang++")
    csrc = os.path.join(ROOT, "paper_2510_12897_amd", "csrc")
    exe = str(tmp_path / "driver")
    subprocess.run([cxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-Wno-unused-function", "-I", os.path.join(ROOT, "include"),
                    "-I", csrc, "-I", os.path.join(ROCM, "include"), "-o", exe,
                    os.path.join(ROOT, "tests", "host", "train_step_driver.cpp"), os.path.join(csrc, "proxy_capi.cpp"),
                    "-L", os.path.join(ROCM, "lib"), f"-Wl,-rpath,{os.path.join(ROCM, 'lib')}", "-lamdhip64"],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr
