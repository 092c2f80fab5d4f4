"""The index arithmetic that kernels and launch plans share (csrc/tq_plan.h), run over its range on the CPU by a small C++
driver (plan_driver.cpp).  No GPU involved."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "driver")
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all", os.path.join(HERE, "plan_driver.cpp"),
                            "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]

    def run(what):
        r = subprocess.run([exe, what], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, (r.stdout + r.stderr)[-2000:]
        return r.stdout

    return run


def test_blocks_of_a_listing_stream_write_every_value_once_and_nothing_else(driver):
    """Blocks that hold no token start (raw values of the block before's last marker) among them."""
    assert "listing streams" in driver("listing")


def test_whole_workgroups_per_matrix_for_every_width(driver):
    """The search for the smallest largest share ends below 8 columns too (an eighth of such a row is no step at all)."""
    assert "cuts" in driver("assign")


def test_cuts_that_the_kernels_multiply_out(driver):
    """Parts of a cost line, bands of a workgroup, pieces of a unit: what the divisions they stand for give."""
    assert "cuts of lines" in driver("cuts")


def test_ring_decode_at_the_distances_it_takes(driver):
    """Lanes exactly as far apart as rings of 128 and of 64 bytes allow, also in segments that end inside a piece."""
    out = driver("ring")
    print(out)
    assert "units decoded" in out


def test_marks_of_units_of_any_lengths_never_share_a_place(driver):
    assert "marks" in driver("marks")


def test_shares_of_units_cut_no_band_twice(driver):
    assert "cut once" in driver("shared")


def test_stages_that_are_cut_by_units(driver):
    """Overlapping outputs, memory that cannot be added to, idle workgroups, bands cut more than once: whole bands then."""
    assert "plans of stages" in driver("stages")
