"""Host-side pieces of the ordering that need no GPU, built with g++ and run here under the address sanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2112_08541_amd", "csrc")


@pytest.mark.parametrize("program", ["order_plan", "order_merge"])
def test_order_program(tmp_path, program):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / program)
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-g", "-Wall", "-Werror", "-fsanitize=address,undefined", "-I" + CSRC,
                           os.path.join(ROOT, "tests", "native", program + ".cpp"), "-o", exe])
    p = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr
    assert p.stdout.startswith("ok"), p.stdout + p.stderr
