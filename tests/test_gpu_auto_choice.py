"""Which kernel CP_PLAN_AUTO takes on both sides of the lane-window plan's rule, told by the launches of a lone t sweep
(the lane-window plan books its launch on the first sweep)."""
import numpy as np
import pytest

from workloads import make_workload

import test_gpu_parity as T

pytestmark = pytest.mark.gpu

gpu = T.gpu


@pytest.mark.parametrize("workload,kw,P,lanes", [
    ("inception", {}, 16, False),                # far reads: a long chain per tick, few partitions to share it
    ("inception", dict(modules=12), 300, False),
    ("inception", {}, 4096, True),
    ("mlp", {}, 16, True),
    ("mlp", {}, 1024, True),
])
def test_lone_t_sweep(gpu, oracle, workload, kw, P, lanes):
    import torch
    w = make_workload(workload, P=P, **kw)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    prof = gpu.CpProfile(1)
    out = gpu.cp_eval(g, a, w.speeds, w.bandwidth, want=("tl",), out_layout=1, profile=prof)
    assert prof.read(0)[1] == ((1, 0) if lanes else (0, 1))
    few = slice(0, min(P, 50))
    ref = oracle.evaluate_workload(w, want=("tl",), threads=8, partitions=few)["tl"]
    assert np.array_equal(out["tl"].cpu().numpy()[few], ref)
    g.close()
