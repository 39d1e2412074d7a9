"""The load rule on keys that carry the device number: both widths of the number, ties, loads that leave the
32 bits of a key within a batch and come back, rows of lanes that are partly used."""
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


@pytest.mark.parametrize("k,speeds_hi,c_hi", [(1, 5, 100), (2, 3, 100), (15, 2, 40), (16, 30, 1000), (17, 30, 1000),
                                              (33, 2, 3), (64, 60, 1000), (16, 4, 2 ** 23), (40, 9, 2 ** 21),
                                              (3, 2, 1)])
@pytest.mark.parametrize("n_last", [1, 63, 64, 65, 900])
def test_seed_on_keys(gpu, oracle, k, speeds_hi, c_hi, n_last):
    rng = np.random.default_rng(k + n_last)
    n, level, src, dst = random_layered_dag(rng, [7, 30, n_last], 1, 3, 2)
    c = rng.integers(0, c_hi, n)
    c[::17] = 0
    w = T._custom("seed-keys", n, src, dst, np.ones(len(src), dtype=np.int64), c, rng.integers(1, speeds_hi + 1, k),
                  np.ones((k, k), dtype=np.int64), np.zeros((1, n), dtype=np.uint8), level)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    got = gpu.cp_seed_partition(g, w.speeds).cpu().numpy()
    assert np.array_equal(got, oracle.seed(w.n, w.succ_ptr, w.succ_idx, w.c, w.speeds, max_len=w.L))
    g.close()
