"""cp_simulate where the state of a partition is kept in LDS: at the edges of each amount kept and of the packed counts."""
import numpy as np
import pytest

from workloads import build_csr, random_layered_dag
from workloads.dags import _finish

import test_gpu_simulate as S

pytestmark = pytest.mark.gpu

gpu = S.gpu


def _case(seed, widths, k, P, inputs, t_hi=100):
    """A layered graph whose last vertex has `inputs` open inputs (or its own, if more)."""
    rng = np.random.default_rng(seed)
    n, level, src, dst = random_layered_dag(rng, widths, 1, 3, 3)
    keep = (dst != n - 1) | (np.cumsum(dst == n - 1) <= inputs)
    src, dst = src[keep], dst[keep]
    more = np.setdiff1d(np.arange(n - widths[-1]), src[dst == n - 1])[:max(0, inputs - int((dst == n - 1).sum()))]
    src, dst = np.concatenate([src, more]), np.concatenate([dst, np.full(len(more), n - 1)])
    csr = build_csr(n, src, dst, rng.integers(1, t_hi, len(src)), level)
    return _finish("resident", csr, rng.integers(1, 60, n), k, rng.integers(1, 20, k), rng.integers(1, 30, (k, k)),
                   rng.integers(0, k, (P, n)).astype(np.uint8))


@pytest.mark.parametrize("inputs", [14, 15, 16, 255, 256])      # 4-bit counts, 8-bit counts, none in LDS
@pytest.mark.parametrize("k,P", [(5, 3), (33, 2), (64, 2), (2, 300)])
def test_packed_counts(gpu, oracle, inputs, k, P):
    S._check(gpu, oracle, _case(inputs + k, [7] * 47 + [3], k, P, inputs), layouts=(0, 1) if P < 10 else (0,))


@pytest.mark.parametrize("n", [1, 7, 8, 9, 8737, 8738, 8739, 9001, 43600, 43800])
def test_sizes_around_each_amount_kept(gpu, oracle, n):
    """Up to 8,738 vertices all of the state of a lone wavefront fits, up to some 43,690 devices and inputs."""
    widths = [n] if n < 20 else [20] * (n // 20) + ([n % 20] if n % 20 else [])
    w = _case(n, widths, 9, 2, 0 if n < 20 else 9)
    assert w.n == n
    S._check(gpu, oracle, w, layouts=(0,))


def test_wide_rows_64_bit_weights_and_a_bad_device_id(gpu, oracle):
    import torch
    w = _case(5, [60, 70, 80, 90], 50, 700, 40, t_hi=2 ** 29)
    S._check(gpu, oracle, w, a=w.assignments[:4], layouts=(0, 1))
    S._check(gpu, oracle, w, layouts=(0,))
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments.copy()).to("cuda:0")
    a[3, w.n - 1] = 50
    with pytest.raises(ValueError):
        gpu.cp_simulate(g, a, w.speeds, w.bandwidth, S.FIFO)
    g.close()
