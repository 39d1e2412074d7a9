"""The wave-column plan at every way its slices are dealt to the XCDs, and the path's search for its start."""
import numpy as np
import pytest

from workloads import random_layered_dag

import test_gpu_parity as T

pytestmark = pytest.mark.gpu

gpu = T.gpu


def _case(seed, widths, k, P):
    rng = np.random.default_rng(seed)
    n, level, src, dst = random_layered_dag(rng, widths, 1, 4, 2)
    hub = np.flatnonzero(level == 1)[:1]                # rows of several sub-rows in both directions
    src = np.concatenate([src, np.full(widths[2], hub[0]), np.flatnonzero(level == 0)])
    dst = np.concatenate([dst, np.flatnonzero(level == 2), np.full(widths[0], hub[0])])
    return T._custom("edges", n, src, dst, rng.integers(0, 90, len(src)), rng.integers(0, 50, n), rng.integers(1, 9, k),
                     rng.integers(1, 20, (k, k)), rng.integers(0, k, (P, n), dtype=np.uint8), level)


@pytest.mark.parametrize("P", [1, 63, 64, 65, 129, 256, 300, 510, 512, 513, 640, 1024, 1030, 1100])
def test_slices_of_64_partitions(gpu, oracle, P):
    T._check(gpu, oracle, _case(P, [37, 5, 130, 1, 3], 5, P), plans=(T.COLUMN,), layouts=(0, 1))


@pytest.mark.parametrize("sources", [1, 255, 256, 257, 511, 512, 513, 2048, 2049, 5000])
def test_start_of_the_path_among_many_sources(gpu, oracle, sources):
    T._check_paths(gpu, oracle, _case(sources, [sources, 4, 6, 2], 3, 5))
