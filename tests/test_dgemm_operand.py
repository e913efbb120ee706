"""Where the FP64 GEMM tiles' direct loads read, checked on the host over rows,
inner lengths, tile edges and leading dimensions."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2510_04795_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_direct_loads_stay_inside_the_matrix(tmp_path):
    exe = str(tmp_path / "dgemm_operand_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, "-o", exe,
                    os.path.join(HERE, "native", "dgemm_operand_check.cpp")], check=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout
    assert p.stdout.startswith("ok ")
