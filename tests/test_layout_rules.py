"""The library's layout rules on the CPU, at sizes no GPU test loads
(tests/layout_rules_driver.cpp over the library's own header)."""
import os
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]
ROCM = "/opt/rocm/include"


def test_layout_rules(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(f"{ROCM}/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers not found")
    exe = tmp_path / "rules"
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-w", "-I", ROCM, "-I", str(ROOT / "include"),
                    "-I", str(ROOT / "paper_1904_02241_amd" / "csrc"),
                    str(ROOT / "tests" / "layout_rules_driver.cpp"), "-o", str(exe)], check=True, timeout=120)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "fails 0" in run.stdout, run.stdout
