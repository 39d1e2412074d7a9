"""A profile names the plan that ran: the one asked for, or what CP_PLAN_AUTO made of the call and its workspace."""
import numpy as np
import pytest

import test_gpu_parity as T
from workloads import make_workload, random_layered_dag

pytestmark = pytest.mark.gpu

gpu = T.gpu


def test_plans_by_name(gpu):
    import torch
    w = make_workload("mlp", P=600)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    prof = gpu.CpProfile(8)
    with pytest.raises(gpu.CpError):
        prof.plan(0)                             # no call yet
    plans = (gpu.PLAN_WAVE_COLUMN, gpu.PLAN_RESIDENT_WINDOW, gpu.PLAN_SHARED_WINDOW_2, gpu.PLAN_LANE_WINDOW)
    for i, plan in enumerate(plans):
        gpu.cp_eval(g, a, w.speeds, w.bandwidth, plan=plan, out_layout=1, profile=prof)
        assert prof.plan(i) == plan
    g.close()


def test_auto_falls_back_where_the_lane_workspace_does_not_fit(gpu, oracle):
    """Aligned rows of a graph numbered by levels: the plan beside the lanes reads them in place and needs the tables only."""
    import torch
    from paper_1711_01912_amd import binding
    rng = np.random.default_rng(4)
    n, level, src, dst = random_layered_dag(rng, [40] * 60, 1, 4, 3)
    P = 64
    w = T._custom("auto", n, src, dst, rng.integers(0, 300, len(src)), rng.integers(0, 50, n), rng.integers(1, 9, 5),
                  rng.integers(1, 20, (5, 5)), rng.integers(0, 5, (P, n), dtype=np.uint8), level)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    ref = oracle.evaluate_workload(w, threads=8)
    stands_for = binding.choose_plan(g, P, w.speeds, w.bandwidth)
    assert stands_for not in (gpu.PLAN_LANE_WINDOW, gpu.PLAN_WAVE_COLUMN)
    prof = gpu.CpProfile(2)
    full = binding.workspace_bytes(g, P, w.k, out_layout=1)
    lanes = binding.workspace_bytes(g, P, w.k, plan=gpu.PLAN_LANE_WINDOW, out_layout=1)
    for i, (size, plan) in enumerate(((full, gpu.PLAN_LANE_WINDOW), (lanes - 256, stands_for))):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda:0")
        out = gpu.cp_eval(g, a, w.speeds, w.bandwidth, out_layout=1, workspace=ws, profile=prof)
        assert prof.plan(i) == plan
        for key in ("cp", "b", "tl"):
            assert np.array_equal(out[key].cpu().numpy(), ref[key]), (key, plan)
    g.close()
