"""Batches of more partitions than one workgroup clears: CP starts from zero in every one of them."""
import numpy as np
import pytest

import test_gpu_parity as T
from workloads import random_layered_dag

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1711_01912_amd as cpe
    cpe.load_library()
    return cpe


@pytest.mark.parametrize("P", [255, 513, 70001, 2048 * 256 + 5])
def test_cp_of_every_partition(gpu, oracle, P):
    import torch
    rng = np.random.default_rng(P)
    n, level, src, dst = random_layered_dag(rng, [2] * 3, 1, 2, 2)
    w = T._custom("huge", n, src, dst, rng.integers(0, 30, len(src)), rng.integers(0, 9, n), [1, 2], [[1, 3], [2, 1]],
                  rng.integers(0, 2, (P, n), dtype=np.uint8), level)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    ref = oracle.evaluate_workload(w, want=("cp",), threads=8)["cp"]
    a = torch.from_numpy(w.assignments).to("cuda:0")
    for plan in (gpu.PLAN_AUTO, gpu.PLAN_WAVE_COLUMN):
        out = {"cp": torch.full((P,), 2 ** 40, dtype=torch.int64, device="cuda:0")}
        gpu.cp_eval(g, a, w.speeds, w.bandwidth, want=("cp", "b"), plan=plan, out=out)
        assert np.array_equal(out["cp"].cpu().numpy(), ref), plan
    g.close()
