"""The quantizer's division in fp32: taken only where it gives the fp64 division's whole number, and by nearly every
wave (a wave of which one lane declines divides in fp64 as a whole)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_fp32_quotient_is_exact_and_taken_by_whole_waves(tmp_path):
    exe = str(tmp_path / "quotient")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I",
                           os.path.join(ROOT, "paper_1812_09162_amd", "csrc"),
                           os.path.join(ROOT, "tests", "quotient_driver.cpp"), "-o", exe])
    waves, slow, slow_rcp, wrong, whole, edges = map(int, subprocess.check_output([exe]).split())
    assert waves == 12_000 and edges == 1
    assert wrong == 0 and whole == 0
    # a quotient is within 2 * slack * x of a whole number by chance: at most 64 * 2 * 256 * 6e-7 = 2 % of the waves
    assert slow < waves * 0.02 and slow_rcp < waves * 0.02, (slow, slow_rcp)
