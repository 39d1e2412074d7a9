"""The rules and tables that the entry points build on the host, compiled by themselves with g++ (no GPU)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from test_packer_sanitized import _deep, _dump
from workloads import build_csr, make_workload, random_layered_dag
from workloads.dags import _finish

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


def test_wave_column_blocks_cover_the_rows_and_leave_long_ones_in_order(harness):
    _holds(harness, "column")


def test_where_calls_with_64_bit_ring_words_end(harness):
    _holds(harness, "wide words")


def test_quotients_by_tables_of_inverses_are_exact(harness):
    _holds(harness, "inverses")


def test_which_walks_are_streamed(harness):
    _holds(harness, "streams")


def test_where_a_few_partitions_take_records(harness):
    _holds(harness, "few records")


def test_left_over_buckets_are_shared_out_over_the_gpu(harness):
    _holds(harness, "left-over")


def test_bins_hold_the_buckets_in_use(harness):
    _holds(harness, "bucket-sizes")


@pytest.mark.parametrize("case", ["tiny", "mlp", "inception", "hubs", "sparse", "deep", "wide-weights"])
def test_blob_is_allocated_once(harness, tmp_path, case):
    if case == "hubs":
        w = make_workload("comm_heavy", P=1, levels=5, width=600, hub_degree=300)
    elif case == "sparse":
        w = make_workload("large_sparse", P=1, levels=150, width=200)
    elif case == "deep":
        w = _deep(0)
    else:
        w = make_workload("tiny" if case == "wide-weights" else case, P=1)
        if case == "wide-weights":
            w.c = w.c * 2**36
    _dump(w, str(tmp_path))
    _holds(harness, "room", str(tmp_path))


@pytest.mark.parametrize("widths,deg,span,wanted", [
    ([30] * 260, 3, 4, "records+jumps"),
    ([1] * 256, 1, 1, "records+jumps"),
    ([30] * 255, 3, 4, "csr+jumps"),
    ([30] * 127, 3, 4, "csr"),
    ([10] * 260, 20, 4, "csr+jumps"),            # rows longer than a record
    ([30] * 260, 3, 200, "csr"),                 # paths of a dozen vertices
])
def test_long_paths_only_by_records_and_jumps(harness, tmp_path, widths, deg, span, wanted):
    rng = np.random.default_rng(len(widths) + span)
    n, level, src, dst = random_layered_dag(rng, widths, 1, deg, span)
    csr = build_csr(n, src, dst, rng.integers(1, 100, len(src)), level)
    w = _finish("paths", csr, rng.integers(1, 60, n), 2, np.ones(2), np.ones((2, 2)), np.zeros((1, n), dtype=np.uint8))
    _dump(w, str(tmp_path))
    _holds(harness, "paths", str(tmp_path), wanted)
