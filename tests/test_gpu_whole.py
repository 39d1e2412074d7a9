"""Small graphs in one launch (CP_PLAN_WHOLE), against the oracle: one vertex, no edges, rows of many units, levels of several
ticks, partitions that do not fill a group or a mask byte, tables with the launch and in memory, the status written by the
launch and cleared before it, 64-bit words, single outputs."""
import numpy as np
import pytest

import test_gpu_parity as T
from workloads import random_layered_dag

pytestmark = pytest.mark.gpu

gpu = T.gpu


def _graph(seed, widths, deg, span, P, k, max_t=1000, max_c=200, hub=0):
    rng = np.random.default_rng(seed)
    n, level, src, dst = random_layered_dag(rng, widths, 1, deg, span)
    if hub:                                      # the first vertex feeds `hub` vertices of the second level
        src = np.concatenate([src, np.zeros(hub, dtype=np.int64)])
        dst = np.concatenate([dst, rng.integers(widths[0], widths[0] + widths[1], hub)])
    return T._custom("whole", n, src, dst, rng.integers(0, max_t, len(src)), rng.integers(0, max_c, n),
                     rng.integers(1, 9, k), rng.integers(1, 60, (k, k)), rng.integers(0, k, (P, n), dtype=np.uint8), level)


def _check(gpu, oracle, w, layout, tick_bytes=None, assign_layout=0, shift=0, whole=True):
    import torch
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = w.assignments if assign_layout == 0 else np.ascontiguousarray(w.assignments.T)
    room = torch.zeros(a.size + shift, dtype=torch.uint8, device="cuda:0")
    room[shift:] = torch.from_numpy(a.ravel())
    a = room[shift:].view(*a.shape)
    ref = oracle.evaluate_workload(w, threads=8)
    prof = gpu.CpProfile(4)
    kw = dict(out_layout=layout, tick_bytes=tick_bytes, assign_layout=assign_layout, profile=prof)
    out = gpu.cp_eval(g, a, w.speeds, w.bandwidth, **kw)
    rows = (lambda x: x.cpu().numpy()) if layout == 1 else (lambda x: x.cpu().numpy().T)
    assert np.array_equal(out["cp"].cpu().numpy(), ref["cp"])
    for key in ("b", "tl"):
        assert np.array_equal(rows(out[key]).astype(np.int64), ref[key]), key
    mask = out["mask"].cpu().numpy().view(np.uint64)
    bits = ref["mask"] if layout == 1 else ref["mask"].T
    assert mask.shape == (bits.shape[0], (bits.shape[1] + 63) // 64)
    padded = np.zeros((bits.shape[0], mask.shape[1] * 64), dtype=bool)           # (bits past the last one are 0)
    padded[:, :bits.shape[1]] = bits
    assert np.array_equal(np.unpackbits(mask.view(np.uint8).reshape(bits.shape[0], -1), axis=1, bitorder="little"), padded)
    for want in ("b", "tl"):
        one = gpu.cp_eval(g, a, w.speeds, w.bandwidth, want=(want,), **kw)
        assert np.array_equal(rows(one[want]).astype(np.int64), ref[want]), want
    one = gpu.cp_eval(g, a, w.speeds, w.bandwidth, want=("cp",), **kw)
    assert np.array_equal(one["cp"].cpu().numpy(), ref["cp"])
    if whole is not None:
        assert (prof.plan(0) == gpu.PLAN_WHOLE) == whole
    g.close()


CASES = {
    "one vertex": dict(widths=[1], deg=1, span=1, P=3, k=2),
    "no edges": dict(widths=[70], deg=1, span=1, P=9, k=1),
    "a chain": dict(widths=[1] * 40, deg=1, span=1, P=1, k=3),
    "eight by eight": dict(widths=[8] * 8, deg=3, span=2, P=16, k=2),
    "a tick and one unit": dict(widths=[9, 17, 33, 65] * 3, deg=1, span=1, P=8, k=5),
    "rows of many units": dict(widths=[20, 100, 20], deg=9, span=2, P=70, k=8, hub=300),
    "a level of many ticks": dict(widths=[300, 3, 300], deg=3, span=2, P=65, k=4),
    "tables with the launch, at most": dict(widths=[20] * 10, deg=3, span=3, P=17, k=29),
    "tables in memory": dict(widths=[20] * 10, deg=3, span=3, P=17, k=30),
    "most devices": dict(widths=[20] * 10, deg=3, span=3, P=5, k=64),
    "64 KB of ids": dict(widths=[16] * 16, deg=3, span=3, P=256, k=7),
    "more": dict(widths=[16] * 16, deg=3, span=3, P=257, k=7),
    "64 lanes, 16 KB of ids": dict(widths=[4] * 8, deg=2, span=2, P=512, k=7),
    "64 lanes, more": dict(widths=[4] * 8, deg=2, span=2, P=513, k=7),
    "several workgroups a unit": dict(widths=[16] * 12, deg=3, span=3, P=5000, k=7),
    "groups of four only": dict(widths=[34] * 60, deg=3, span=3, P=1024, k=60),
    "too many vertices": dict(widths=[1] * 2049, deg=1, span=1, P=8, k=2),
}


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("case", CASES)
def test_against_the_oracle(gpu, oracle, case, layout):
    _check(gpu, oracle, _graph(3, **CASES[case]), layout, whole={"groups of four only": None, "too many vertices": False}.get(case, True))


@pytest.mark.parametrize("kw,tick_bytes", [
    (dict(max_t=1 << 28, max_c=1 << 20), None),                  # paths past 32 bits
    (dict(max_t=1 << 22, max_c=1 << 20), None),                  # ring words of 64 bits, ticks of 32
    (dict(), 8),                                                 # 32-bit words, 64-bit outputs
])
@pytest.mark.parametrize("layout", [0, 1])
def test_wide_ticks(gpu, oracle, kw, tick_bytes, layout):
    _check(gpu, oracle, _graph(5, [10, 30] * 12, 4, 6, 19, 6, **kw), layout, tick_bytes)


@pytest.mark.parametrize("shift", [0, 1, 4])
@pytest.mark.parametrize("assign_layout", [0, 1])
def test_ids_by_vertex_and_out_of_line(gpu, oracle, assign_layout, shift):
    for layout in (0, 1):
        _check(gpu, oracle, _graph(6, [13] * 9, 3, 3, 21, 5), layout, assign_layout=assign_layout, shift=shift)


@pytest.mark.parametrize("P", [3, 20, 700])
@pytest.mark.parametrize("shift", [0, 1])
def test_a_device_id_too_large_is_reported(gpu, P, shift):
    import torch
    w = _graph(9, [13] * 9, 3, 4, P, 4)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    room = torch.zeros(P * w.n + shift, dtype=torch.uint8, device="cuda:0")
    a = room[shift:].view(P, w.n)
    for q, v in ((0, 0), (P - 1, w.n - 1), (P // 2, 50)):
        a[:] = torch.from_numpy(w.assignments)
        a[q, v] = 4
        with pytest.raises(ValueError):
            gpu.cp_eval(g, a, w.speeds, w.bandwidth, out_layout=1)
        a[q, v] = 0
        gpu.cp_eval(g, a, w.speeds, w.bandwidth, out_layout=1)
    g.close()
