"""cp_simulate with owners and inputs in LDS (from 8,739 vertices on), the first vertices handed over in a step too (from 513
partitions on): as many vertices handed to one device in a step as wait in LDS, one fewer and more, by a short row, by a
row the whole wavefront shares, and at the start."""
import numpy as np
import pytest

from workloads import build_csr
from workloads.dags import _finish

import test_gpu_simulate as S

pytestmark = pytest.mark.gpu

gpu = S.gpu


@pytest.mark.parametrize("handed", [1, 2, 3, 4, 5, 31, 40])
@pytest.mark.parametrize("k", [3, 33, 64])
def test_vertices_handed_over_in_one_step(gpu, oracle, handed, k):
    _handed_over(gpu, oracle, handed, k, 1)


@pytest.mark.parametrize("handed,k", [(1, 3), (2, 33), (3, 64), (5, 3), (31, 33), (40, 64)])
def test_the_same_in_a_batch_with_near_inboxes(gpu, oracle, handed, k):
    _handed_over(gpu, oracle, handed, k, 257)


def _handed_over(gpu, oracle, handed, k, copies):
    rng = np.random.default_rng(handed + k)
    roots, lone = 40, 8800                       # vertices without edges: sources that start on every device
    src = np.repeat(np.arange(roots), handed)
    dst = roots + np.arange(roots * handed)
    n = roots + roots * handed + lone
    level = np.zeros(n, dtype=np.int64)
    level[dst] = 1
    csr = build_csr(n, src, dst, rng.integers(1, 100, len(src)), level)
    a = rng.integers(0, k, (2, n)).astype(np.uint8)
    a[0, dst] = np.repeat(rng.integers(0, k, roots), handed)        # a root's successors on one device
    a[1, n - lone:] = k - 1
    a = np.tile(a, (copies, 1))
    w = _finish("inbox", csr, rng.integers(1, 60, n), k, rng.integers(1, 20, k), rng.integers(1, 30, (k, k)), a)
    S._check(gpu, oracle, w, layouts=(0,))
