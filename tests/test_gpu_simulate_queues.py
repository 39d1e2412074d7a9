"""cp_simulate where queues outgrow the keys in registers and out-degrees what a vertex's record holds."""
import numpy as np
import pytest

from workloads import build_csr
from workloads.dags import _finish

import test_gpu_simulate as S

pytestmark = pytest.mark.gpu

gpu = S.gpu


def _stars(seed, stars, leaves, k, P, t_hi=100):
    """`stars` vertices without predecessors, of 0 to `leaves` out-edges each, to `leaves` shared heads that feed one sink."""
    rng = np.random.default_rng(seed)
    degree = np.arange(stars) % (leaves + 1)
    src = np.repeat(np.arange(stars), degree)
    dst = stars + np.concatenate([rng.permutation(leaves)[:d] for d in degree])
    heads = np.unique(dst)
    n = stars + leaves + 1
    src, dst = np.concatenate([src, heads]), np.concatenate([dst, np.full(len(heads), n - 1)])
    level = np.concatenate([np.zeros(stars, np.int64), np.ones(leaves, np.int64), [2]])
    csr = build_csr(n, src, dst, rng.integers(1, t_hi, len(src)), level)
    return _finish("stars", csr, rng.integers(1, 60, n), k, rng.integers(1, 20, k), rng.integers(1, 30, (k, k)) * max(1, t_hi >> 8),
                   rng.integers(0, k, (P, n)).astype(np.uint8))


@pytest.mark.parametrize("leaves", [1, 2, 3, 4, 5, 8, 9, 31, 33])       # 3: the most a record holds; 32: a wide row
@pytest.mark.parametrize("k,P", [(1, 8), (2, 700), (33, 9), (2, 7)])    # state all in LDS, shared by many, few vertices a device; no records
def test_rows_around_what_a_record_holds(gpu, oracle, leaves, k, P):
    S._check(gpu, oracle, _stars(leaves, leaves + 1, leaves, k, P), layouts=(0, 1) if P < 10 else (0,))


@pytest.mark.parametrize("stars", [1, 2, 3, 4, 5, 6, 20, 90])           # three keys of a queue lie in registers
@pytest.mark.parametrize("k", [1, 3])
def test_queues_around_what_registers_hold(gpu, oracle, stars, k):
    S._check(gpu, oracle, _stars(100 + stars, stars, 6, k, 4), layouts=(0,))


def test_64_bit_weights_have_no_records(gpu, oracle):
    S._check(gpu, oracle, _stars(7, 20, 9, 4, 12, t_hi=2 ** 40), layouts=(0, 1))


def test_priorities_out_of_range_are_reported_from_registers_and_memory(gpu, oracle):
    import torch
    w = _stars(9, 40, 6, 2, 3)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    for v in (0, 39, w.n - 1):
        for value in (-1, 2 ** 31, 2 ** 32, 2 ** 33 + 5):
            b = torch.ones((3, w.n), dtype=torch.int64, device="cuda:0")
            b[1, v] = value
            with pytest.raises(ValueError):
                gpu.cp_simulate(g, a, w.speeds, w.bandwidth, S.PCT, b=b, b_layout=1)
    g.close()
