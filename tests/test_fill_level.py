"""The fill level of a shared buffer between two steps that add to it: every thread of a block reads the same one, however late
it leaves the barrier before (the oracle without the second barrier does not)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_late_thread_reads_the_same_level(tmp_path):
    exe = str(tmp_path / "fill_level")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_1812_09162_amd", "csrc"),
                           os.path.join(ROOT, "tests", "fill_level_driver.cpp"), "-o", exe])
    kept, one_barrier = map(int, subprocess.check_output([exe], timeout=60).split())
    assert kept == 0
    assert one_barrier > 0  # the model does tell them apart
