"""The load rule's batches: counts of vertices to be placed around multiples of 8 and 64, one, two and four devices per
lane, batches whose loads are keys, 32 bits and 64 bits, ties in each of the three between the devices of a lane and of a
row, speeds and costs without multiply-shift constants."""
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


@pytest.mark.parametrize("k,c_hi", [(3, 50), (16, 1000), (31, 1000), (32, 2 ** 20), (48, 1000), (16, 2 ** 25), (5, 2 ** 30),
                                    (32, 2 ** 25), (17, 2 ** 26), (64, 2 ** 24), (48, 2 ** 26), (64, 2 ** 28)])
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


@pytest.mark.parametrize("k", [2, 16, 17, 32, 48, 64])
@pytest.mark.parametrize("c", [7, 2 ** 21, 2 ** 23, 2 ** 25, 2 ** 26 - 1, 2 ** 26, 2 ** 29])
def test_ties(gpu, oracle, k, c):
    """Vertices alike and two speeds only: devices tie all the time, the lowest has to win whatever form the loads have; 2^23
    and 2^25 need 32 bits (2^26 - 1 the last of them), 2^26 more."""
    rng = np.random.default_rng(k)
    n, level, src, dst = random_layered_dag(rng, [1, 1, 777], 1, 1, 1)
    cs = np.full(n, c)
    cs[rng.random(n) < 0.1] = c // 2
    w = T._custom("seed-ties", n, src, dst, np.ones(len(src), dtype=np.int64), cs, 2 + np.arange(k) % 2,
                  np.ones((k, k), dtype=np.int64), np.zeros((1, n), dtype=np.uint8), level)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    got = gpu.cp_seed_partition(g, w.speeds).cpu().numpy()
    assert np.array_equal(got, oracle.seed(w.n, w.succ_ptr, w.succ_idx, w.c, w.speeds, max_len=w.L))
    g.close()
