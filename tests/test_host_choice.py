"""The estimate by which a launch goes to the ring kernel or the runs kernel (csrc/tq_choice.h): the longest share against all
workgroups one by one, its growth with the work, and launches that were timed on both kernels (choice_driver.cpp).  No GPU involved."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_estimate_of_the_batched_kernels_times(tmp_path):
    exe = str(tmp_path / "driver")
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                            os.path.join(HERE, "choice_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-2000:]
