"""Lines of the size rules in rules.h, without a GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "rules")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1812_09162_amd", "csrc"),
                           os.path.join(ROOT, "tests", "rules_driver.cpp"), "-o", exe])

    def ask(name, *args):
        line = " ".join(map(str, (name, *args, *[0] * (5 - len(args)))))
        return int(subprocess.check_output([exe], input=line.encode()))
    return ask


@pytest.mark.parametrize("nq,per_query,calibration,pilot,cheap,wide", [
    (1, 1, 400, 0, 1, 1), (256, 1, 400, 0, 0, 1), (257, 1, 400, 0, 1, 0), (512, 1, 4000, 0, 0, 0),  # one block a query: up to one a CU
    (257, 1, 400, 4096, 1, 1), (512, 1, 400, 6400, 0, 1), (513, 1, 400, 6400, 0, 0),                # ... with a pilot two
    (1, 128, 400, 65536, 1, 0), (1, 128, 1024, 65536, 0, 0),                                        # short calibrations beside scans
    (1, 128, 1028, 65536, 1, 1), (2, 128, 2048, 65536, 0, 1), (3, 128, 1028, 65536, 0, 0), (4, 128, 2048, 65536, 0, 0),
    (4, 128, 4000, 65536, 1, 0), (4, 128, 2052, 65536, 0, 1), (4, 128, 8000, 65536, 1, 1), (5, 128, 8000, 65536, 0, 0),
])
def test_width_of_the_quantizers_blocks(rule, nq, per_query, calibration, pilot, cheap, wide):
    assert rule("quantize_wide", nq * per_query, per_query, calibration, pilot, cheap) == wide


@pytest.mark.parametrize("nq,threads", [(1, 1024), (256, 1024), (257, 512), (512, 512), (513, 256)])
def test_width_of_the_calibrations_blocks(rule, nq, threads):
    assert rule("calib_threads", nq) == threads


@pytest.mark.parametrize("n,R,nq,codes", [
    (10_000_000, 1000, 1, 1_024_000), (4_096_000, 1000, 4, 1_024_000), (3_000_000, 1000, 1, 750_000), (2_048_000, 1000, 1, 512_000),
    (1_000_000, 1000, 2, 512_000), (1, 2048, 1, 1_048_576), (10_000_000, 1000, 5, 512_000), (10_000_000, 2048, 512, 1_048_576)])
def test_pilot_for_long_results(rule, n, R, nq, codes):
    assert rule("pilot_for_results", n, R, nq) == codes  # few queries: up to 1024 a result, a quarter of the list; else 512


@pytest.mark.parametrize("pairs,cells,shared", [
    (1023, 256, 0), (1024, 256, 1), (1536, 1024, 1), (1535, 1024, 0), (640_000, 65_536, 1), (64_000, 65_536, 0),
    (1200, 100, 0), (2000, 100, 0), (3520, 100, 1), (2048, 64, 0), (4096, 64, 1),  # too few groups for the CUs
])
def test_when_pairs_share_a_pass_over_a_list(rule, pairs, cells, shared):
    assert rule("ivf_shared_pays", pairs, cells) == shared


@pytest.mark.parametrize("nq,n,nibbles,blocks", [
    (1, 10_000_000, 1, 2048), (2, 10_000_000, 1, 1024), (16, 100_000_000, 1, 1024), (1, 1 << 24, 0, 1024), (1, (1 << 24) + 1, 0, 2048)])
def test_blocks_of_the_look_up_scan(rule, nq, n, nibbles, blocks):
    assert rule("scan_blocks_most", nq, n, nibbles) == blocks


def test_header_states_the_lines_of_the_shared_pass():
    text = " ".join(open(os.path.join(ROOT, "include", "qadc.h")).read().replace("*", " ").split())
    assert text.count("1.5 pairs per cell, 1024 pairs and K + pairs / 16 >= 320") == 1
    assert text.count("1.5 (query, probe) pairs per cell, 1024 pairs and K + pairs / 16 >= 320") == 1
