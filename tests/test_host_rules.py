"""The rules and tables that the entry points build on the host, compiled by themselves with g++ (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_01912_amd", "csrc")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    out = tmp_path_factory.mktemp("rules") / "harness"
    cmd = ["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           os.path.join(ROOT, "tests", "host_rules_harness.cpp"), os.path.join(CSRC, "graph.cpp"),
           os.path.join(CSRC, "cost.cpp"), "-o", str(out)]
    subprocess.run(cmd, check=True)
    return str(out)


def _holds(harness, *args):
    run = subprocess.run([harness, *args], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout + run.stderr


def test_large_batches_are_cleared_by_as_many_threads(harness):
    _holds(harness, "prepare")


def test_wave_column_blocks_cover_the_rows_and_share_long_ones_out(harness):
    _holds(harness, "column")


def test_rounded_cost_tables_are_exact_and_built_only_on_request(harness):
    _holds(harness, "rounded")
