"""Units whose lanes run too far apart for a ring, as the device gets them: the same bytes in the same number of chunks, the
lanes no further apart than the limit (level_driver.cpp).  No GPU involved."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2509_22951_amd as tq
from drifting import lane_reach

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_units_are_brought_together(tmp_path):
    exe = str(tmp_path / "driver")
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-pthread",
                            os.path.join(HERE, "level_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, (r.stdout + r.stderr)[-2000:]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("lmax,pad", [(2, 1), (3, 4)])
def test_lanes_reach_a_column_further_with_every_pad(lmax, pad):
    """Rows of zeros next to rows without a pair: the zero rows' lanes end after half (lmax 3: a third) of the codes.  A pad is a single
    byte on the device, and counts four times where runs may be longer than 2 bytes."""
    Q = np.zeros((32, 256), np.int8)
    Q[17::2] = np.resize(np.arange(1, 114, dtype=np.int8), 8 * 256).reshape(8, 256)
    blob = tq.tq_encode_quantized(Q, np.ones(32, np.float32), max_entries=256 + lmax - 1, seg_cols=64, lmax=lmax)
    info = tq.tq_validate_blob(blob)
    assert info["n_entries"] == 256 + lmax - 1
    steps = 64                                  # codes of a lane of single bytes: the second band's units
    short = -(-64 // lmax)                      # of a lane of zeros
    assert lane_reach(blob) == 64 + pad * (steps - short)
