"""The wave-column plan where it goes slice by slice: thousands of rows, an odd number of 64-partition slices."""
import numpy as np
import pytest

import test_gpu_parity as T
from workloads import random_layered_dag

pytestmark = pytest.mark.gpu

gpu = T.gpu


@pytest.mark.parametrize("tick_bytes,P", [(4, 1025), (4, 1088), (8, 570)])
def test_rows_of_every_length_slice_by_slice(gpu, oracle, tick_bytes, P):
    from gpu_util import assert_equal_to_oracle, run_gpu
    rng = np.random.default_rng(P)
    n, level, src, dst = random_layered_dag(rng, [3001, 3006, 40], 1, 4, 2)
    hub = np.flatnonzero(level == 1)[0]          # a row of 3,001 edges beside them
    src = np.concatenate([src, np.flatnonzero(level == 0)])
    dst = np.concatenate([dst, np.full(3001, hub)])
    w = T._custom("order", n, src, dst, rng.integers(0, 90, len(src)), rng.integers(0, 50, n), rng.integers(1, 9, 5),
                  rng.integers(1, 20, (5, 5)), rng.integers(0, 5, (P, n), dtype=np.uint8), level)
    res = run_gpu(w, T.COLUMN, tick_bytes=tick_bytes)
    assert_equal_to_oracle(res, oracle.evaluate_workload(w, threads=8), f"P {P}")
