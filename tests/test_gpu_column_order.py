"""The wave-column plan in its two orders: hub rows and long rows in runs, slice by slice, the others row by row."""
import numpy as np
import pytest

import test_gpu_parity as T
from workloads import random_layered_dag

pytestmark = pytest.mark.gpu

gpu = T.gpu


@pytest.mark.parametrize("degree", [63, 64, 200, 255, 256, 700])      # around a long row and a hub row
@pytest.mark.parametrize("tick_bytes,P", [(4, 1), (4, 130), (4, 260), (4, 500), (8, 570), (4, 1088)])
def test_rows_of_every_length(gpu, oracle, degree, tick_bytes, P):
    from gpu_util import assert_equal_to_oracle, run_gpu
    rng = np.random.default_rng(P + degree)
    n, level, src, dst = random_layered_dag(rng, [150, 701, 43], 1, 4, 2)
    first, mid, last = (np.flatnonzero(level == x) for x in range(3))
    wide = [first[0], first[7], mid[3]]                    # long rows in both directions
    ends = [rng.choice(mid, degree - 4), rng.choice(mid, degree - 4), rng.choice(last, degree - 4)]
    src = np.concatenate([src, *[np.full(len(e), v) for v, e in zip(wide, ends)], rng.choice(mid, degree)])
    dst = np.concatenate([dst, *ends, np.full(degree, last[5])])
    w = T._custom("order", n, src, dst, rng.integers(0, 90, len(src)), rng.integers(0, 50, n), rng.integers(1, 9, 5),
                  rng.integers(1, 20, (5, 5)), rng.integers(0, 5, (P, n), dtype=np.uint8), level)
    res = run_gpu(w, T.COLUMN, tick_bytes=tick_bytes)
    assert_equal_to_oracle(res, oracle.evaluate_workload(w, threads=8), f"P {P} degree {degree}")
