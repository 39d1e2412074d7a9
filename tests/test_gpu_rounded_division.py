"""Divisions as one multiply-add rounded up (lane-window and whole-graph plans, and the resident-window plan's transfers of 16-bit
volumes; the wave-column plan's: test_gpu_column4.py), against the oracle: volumes at and around multiples of the divisors, up to and past the last volume that floats hold (2^23 - 1), divisors from 1 to far above it."""
import numpy as np
import pytest

import test_gpu_parity as T
from workloads import random_layered_dag

pytestmark = pytest.mark.gpu

gpu = T.gpu

DIVISORS = np.array([1, 2, 3, 5, 7, 10, 255, 256, 257, 4095, 65537, 2**20 + 7, 2**22 + 1, 2**23 - 1, 2**23, 2**24 + 1,
                     2**30 + 3, 2**31 - 2**24 - 1])


def _volumes(rng, count, top):
    d = rng.choice(DIVISORS, count)
    x = rng.integers(0, top + 1, count) // d * d + rng.integers(-1, 2, count)
    x[rng.integers(0, count, 8)] = top
    x[rng.integers(0, count, 8)] = 0
    return np.clip(x, 0, top)


@pytest.mark.parametrize("plan", ["PLAN_AUTO", "PLAN_LANE_WINDOW"])
@pytest.mark.parametrize("top", [1, 10_000, 2**23 - 1, 2**23, 2**24 - 1, 2**24, 2**30])
def test_against_the_oracle(gpu, oracle, top, plan):
    import torch
    rng = np.random.default_rng(top)
    k, P = len(DIVISORS), 8
    n, level, src, dst = random_layered_dag(rng, [30] * 8, 1, 4, 2)
    w = T._custom("division", n, src, dst, _volumes(rng, len(src), top), _volumes(rng, n, top), rng.permutation(DIVISORS),
                  rng.choice(DIVISORS, (k, k)), rng.integers(0, k, (P, n), dtype=np.uint8), level)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    ids = torch.from_numpy(w.assignments).to("cuda:0")
    ref = oracle.evaluate_workload(w, threads=8)
    for layout in (0, 1):
        out = gpu.cp_eval(g, ids, w.speeds, w.bandwidth, out_layout=layout, plan=getattr(gpu, plan))
        assert np.array_equal(out["cp"].cpu().numpy(), ref["cp"])
        for key in ("b", "tl"):
            rows = out[key].cpu().numpy()
            assert np.array_equal((rows if layout == 1 else rows.T).astype(np.int64), ref[key]), (key, layout)
    g.close()


# what multiply-shift constants exist for, which the plan asks for
SHORT_DIVISORS = np.array([1, 2, 3, 5, 7, 10, 63, 64, 65, 255, 256, 257, 4095, 4096, 4097, 30011])


@pytest.mark.parametrize("k", [1, 2, 15, 16, 32, 64])        # rows of transfer costs lie an odd number of words apart
@pytest.mark.parametrize("top", [1, 10_000, 65_535])
def test_16_bit_volumes_of_the_resident_window_plan(gpu, oracle, top, k):
    import torch
    rng = np.random.default_rng([top, k])
    P = 6
    n, level, src, dst = random_layered_dag(rng, [90] * 40, 1, 5, 4)
    d = rng.choice(SHORT_DIVISORS, len(src))
    t = np.clip(rng.integers(0, top + 1, len(src)) // d * d + rng.integers(-1, 2, len(src)), 0, top)
    t[:4] = top
    w = T._custom("division", n, src, dst, t, rng.integers(0, 1000, n), rng.choice(SHORT_DIVISORS, k),
                  rng.choice(SHORT_DIVISORS, (k, k)), rng.integers(0, k, (P, n), dtype=np.uint8), level)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    ids = torch.from_numpy(w.assignments).to("cuda:0")
    ref = oracle.evaluate_workload(w, threads=8)
    for layout in (0, 1):                        # two launches, and both sweeps in one
        prof = gpu.CpProfile(1)
        out = gpu.cp_eval(g, ids, w.speeds, w.bandwidth, out_layout=layout, plan=gpu.PLAN_RESIDENT_WINDOW, profile=prof)
        assert np.array_equal(out["cp"].cpu().numpy(), ref["cp"])
        for key in ("b", "tl"):
            rows = out[key].cpu().numpy()
            assert np.array_equal((rows if layout == 1 else rows.T).astype(np.int64), ref[key]), (key, layout)
    g.close()
