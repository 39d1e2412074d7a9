"""The load rule's batches: counts of vertices to be placed around multiples of 8 and 64, one, two and four devices per
lane, loads that leave the keys for some batches only, speeds and costs without multiply-shift constants."""
import numpy as np
import pytest

from workloads import random_layered_dag

import test_gpu_parity as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1711_01912_amd as cpe
    cpe.load_library()
    return cpe


@pytest.mark.parametrize("k,c_hi", [(3, 50), (16, 1000), (31, 1000), (32, 2 ** 20), (48, 1000), (16, 2 ** 25), (5, 2 ** 30)])
@pytest.mark.parametrize("n_last", [6, 14, 15, 62, 70, 71, 72, 126, 135, 2500])
def test_seed_batches(gpu, oracle, k, c_hi, n_last):
    rng = np.random.default_rng(31 * k + n_last)
    n, level, src, dst = random_layered_dag(rng, [1, 1, n_last], 1, 1, 1)
    c = rng.integers(0, 100, n)
    c[rng.random(n) < 0.05] = c_hi            # few large ones: some batches leave the keys, others come back
    w = T._custom("seed-batches", n, src, dst, np.ones(len(src), dtype=np.int64), c, rng.integers(1, 20, k),
                  np.ones((k, k), dtype=np.int64), np.zeros((1, n), dtype=np.uint8), level)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    got = gpu.cp_seed_partition(g, w.speeds).cpu().numpy()
    assert np.array_equal(got, oracle.seed(w.n, w.succ_ptr, w.succ_idx, w.c, w.speeds, max_len=w.L))
    g.close()
