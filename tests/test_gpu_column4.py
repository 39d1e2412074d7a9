"""The wave-column plan with four partitions a lane (32-bit ticks, batches of a multiple of four) against the oracle: slices that
are not full, rows that do not fill a wavefront, hubs of all lengths, device counts up to the most, volumes next to multiples of
the divisors up to the largest that 32-bit ticks allow."""
import numpy as np
import pytest

import test_gpu_parity as T
from workloads import random_layered_dag

pytestmark = pytest.mark.gpu

gpu = T.gpu


def _check(gpu, oracle, w, layouts=(0, 1), assign_layouts=(0, 1)):
    import torch
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    ref = oracle.evaluate_workload(w, threads=8)
    for layout in layouts:
        for by_vertex in assign_layouts:
            assert w.n // (int(w.level_ptr.shape[0]) - 1) * ((w.P + 63) // 64) >= 10240
            a = torch.from_numpy(np.ascontiguousarray(w.assignments.T) if by_vertex else w.assignments).to("cuda:0")
            out = gpu.cp_eval(g, a, w.speeds, w.bandwidth, plan=gpu.PLAN_WAVE_COLUMN, out_layout=layout,
                              assign_layout=by_vertex)
            rows = (lambda x: x.cpu().numpy()) if layout == 1 else (lambda x: x.cpu().numpy().T)
            for key in ("b", "tl"):
                assert np.array_equal(rows(out[key]), ref[key]), (key, layout, by_vertex)
            assert np.array_equal(out["cp"].cpu().numpy(), ref["cp"])
    g.close()


@pytest.mark.parametrize("P", [4, 60, 68, 256, 516])
@pytest.mark.parametrize("k", [1, 2, 8, 32, 33])
def test_batches_and_devices(gpu, oracle, P, k):
    rng = np.random.default_rng([P, k])
    wide = 10240 // ((P + 63) // 64)              # (the rule asks for that many rows and slices in a level, on average)
    n, level, src, dst = random_layered_dag(rng, [3 * wide, 1, 50, 2 * wide + 3, 17], 1, 5, 3)
    few = np.arange(40)                          # rows of up to 200 edges
    src = np.concatenate([src, np.repeat(few, 5 * few)])
    dst = np.concatenate([dst, rng.integers(3 * wide, n, (5 * few).sum())])
    w = T._custom("column4", n, src, dst, rng.integers(0, 1 << 20, len(src)), rng.integers(0, 1 << 20, n),
                  rng.integers(1, 300, k), rng.integers(1, 300, (k, k)), rng.integers(0, k, (P, n), dtype=np.uint8), level)
    _check(gpu, oracle, w)


@pytest.mark.parametrize("length", [255, 256, 257, 300, 1024, 4097])
def test_hubs(gpu, oracle, length):
    rng = np.random.default_rng(length)
    n, level, src, dst = random_layered_dag(rng, [7, 16000, 40], 1, 4, 2)
    src = np.concatenate([src, np.full(length, 3), rng.integers(7, 16007, length)])    # out of vertex 3, into 16010
    dst = np.concatenate([dst, rng.integers(7, 16007, length), np.full(length, 16010)])
    w = T._custom("column4", n, src, dst, rng.integers(0, 5000, len(src)), rng.integers(0, 500, n), rng.integers(1, 9, 6),
                  rng.integers(1, 60, (6, 6)), rng.integers(0, 6, (72, n), dtype=np.uint8), level)
    _check(gpu, oracle, w)


@pytest.mark.parametrize("most", [1 << 8, 1 << 24, (1 << 30) - 1])
def test_volumes_next_to_multiples(gpu, oracle, most):
    """Two levels, an edge from every vertex of the first: t is a multiple of some divisor, one less or one more."""
    rng = np.random.default_rng(most)
    N, k, P = 10240, 32, 64
    rates = rng.choice(np.concatenate([np.arange(1, 258), 2 ** np.arange(9, 30), [1000003, 2 ** 31 - 1, 2 ** 40]]), (k, k))
    d = rng.choice(rates.ravel(), N)
    t = np.clip(d * np.maximum(1, rng.integers(0, most, N) // d) + rng.integers(-1, 2, N), 0, most)
    c = np.clip(rng.integers(0, most, 2 * N), 0, most)
    w = T._custom("column4", 2 * N, np.arange(N), rng.permutation(N) + N, t, c // 2, rng.choice(rates.ravel(), k), rates,
                  rng.integers(0, k, (P, 2 * N), dtype=np.uint8), np.repeat([0, 1], N))
    _check(gpu, oracle, w, layouts=(1,), assign_layouts=(0,))
