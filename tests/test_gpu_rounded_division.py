"""Divisions as one multiply-add rounded up (lane-window, whole-graph and wave-column plans), against the oracle: volumes at and
around multiples of the divisors, up to and past the last volume that floats hold (2^23 - 1), divisors from 1 to far above it."""
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


@pytest.mark.parametrize("plan", ["PLAN_AUTO", "PLAN_LANE_WINDOW", "PLAN_WAVE_COLUMN"])
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
