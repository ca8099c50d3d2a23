"""Contexts are created and destroyed against a stand-in for the HIP runtime (create_check.cpp), so
what ds_create leaves behind is checked without a GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1905_05957_amd")


def test_create_against_a_stand_in_runtime(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    binary = str(tmp_path / "create_check")
    # -rdynamic: the program's own functions answer for the runtime's
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", os.path.join(HERE, "create_check.cpp"), "-o", binary,
                    "-rdynamic", "-L" + PKG, "-lds_hip", "-Wl,--unresolved-symbols=ignore-in-shared-libs",
                    f"-Wl,-rpath,{PKG}:{rocm}/lib"], check=True)
    r = subprocess.run([binary], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "FAILED" not in r.stdout and "ok: ternary" in r.stdout, r.stdout + r.stderr
