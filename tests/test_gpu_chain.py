"""Sweeps of a few partitions by one workgroup each (CP_PLAN_CHAIN), against the oracle: ticks of one and of several
wavefronts, levels of several ticks, rows longer than a tick, empty levels' worth of padding, edges that reach far back in the
ring, both layouts, 64-bit ticks, plain divisors, single outputs, and the rule's edges."""
import numpy as np
import pytest

import test_gpu_parity as T
from paper_1711_01912_amd import binding
from workloads import random_layered_dag

pytestmark = pytest.mark.gpu

gpu = T.gpu


def _graph(seed, widths, deg, span, P, k, max_t=1000, max_c=200, hubs=0):
    rng = np.random.default_rng(seed)
    n, level, src, dst = random_layered_dag(rng, widths, 1, deg, span)
    if hubs:                                     # a vertex of every 50th level feeds `hubs` vertices of the next one
        first = np.concatenate([[0], np.cumsum(widths)])
        for l in range(0, len(widths) - 1, 50):
            src = np.concatenate([src, np.full(hubs, first[l])])
            dst = np.concatenate([dst, rng.integers(first[l + 1], first[l + 2], hubs)])
    return T._custom("chain", n, src, dst, rng.integers(0, max_t, len(src)), rng.integers(0, max_c, n),
                     rng.integers(1, 9, k), rng.integers(1, 60, (k, k)), rng.integers(0, k, (P, n), dtype=np.uint8), level)


def _check(gpu, oracle, w, layout, tick_bytes=None, chain=True):
    import torch
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    ref = oracle.evaluate_workload(w, threads=8)
    prof = gpu.CpProfile(1)
    out = gpu.cp_eval(g, a, w.speeds, w.bandwidth, out_layout=layout, profile=prof, tick_bytes=tick_bytes)
    assert (prof.plan(0) == gpu.PLAN_CHAIN) == chain
    rows = (lambda x: x.cpu().numpy()) if layout == 1 else (lambda x: x.cpu().numpy().T)
    assert np.array_equal(out["cp"].cpu().numpy(), ref["cp"])
    for key in ("b", "tl"):
        assert np.array_equal(rows(out[key]).astype(np.int64), ref[key]), key
    for key in ("b", "tl"):                      # one sweep alone
        one = gpu.cp_eval(g, a, w.speeds, w.bandwidth, want=(key,), out_layout=layout, tick_bytes=tick_bytes)
        assert np.array_equal(rows(one[key]).astype(np.int64), ref[key]), key
    g.close()


CASES = {
    "one wavefront, levels of one vertex": dict(widths=[1] * 300, deg=1, span=3, P=1, k=2),
    "one wavefront": dict(widths=[30, 1, 2, 17] * 70, deg=4, span=7, P=3, k=5),
    "exactly a tick and one more": dict(widths=[64, 65] * 130, deg=3, span=2, P=2, k=16),
    "several wavefronts": dict(widths=[211] * 260, deg=7, span=10, P=5, k=16),
    "levels of several ticks among narrow ones": dict(widths=([5] * 20 + [1500]) * 13, deg=3, span=1, P=2, k=7),
    "rows longer than a tick": dict(widths=[40] * 300, deg=3, span=4, P=2, k=4, hubs=1500),
    "far back in the ring": dict(widths=[60] * 280, deg=4, span=270, P=2, k=50),
    "more devices than lanes": dict(widths=[25] * 290, deg=3, span=5, P=1, k=80),
    "most partitions": dict(widths=[30] * 300, deg=4, span=4, P=64, k=8),
}


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("case", CASES)
def test_against_the_oracle(gpu, oracle, case, layout):
    _check(gpu, oracle, _graph(3, **CASES[case]), layout)


@pytest.mark.parametrize("kw,tick_bytes", [
    (dict(max_t=1 << 28, max_c=1 << 20), None),                  # paths past 32 bits
    (dict(max_t=(1 << 32) - 300, max_c=200), None),             # no multiply-shift form
    (dict(max_t=65300, max_c=200), None),                        # costs of up to 16 bits, and one more
    (dict(max_t=65600, max_c=200), None),
    (dict(), 8),                                                 # 32-bit paths, 64-bit outputs
])
@pytest.mark.parametrize("layout", [0, 1])
def test_wide_ticks(gpu, oracle, kw, tick_bytes, layout):
    _check(gpu, oracle, _graph(5, [40, 70] * 140, 4, 6, 3, 6, **kw), layout, tick_bytes)


def test_where_the_rule_ends(gpu, oracle):
    """Fewer levels, more partitions, and a ring that LDS cannot hold go another way."""
    _check(gpu, oracle, _graph(7, [30] * 255, 3, 4, 2, 4), 1, chain=False)
    _check(gpu, oracle, _graph(7, [30] * 256, 3, 4, 2, 4), 1)
    _check(gpu, oracle, _graph(7, [30] * 256, 3, 4, 65, 4), 1, chain=False)
    _check(gpu, oracle, _graph(7, [160] * 300, 3, 299, 2, 4), 1, chain=False)


def test_a_device_id_too_large_is_reported(gpu):
    import torch
    w = _graph(9, [30] * 300, 3, 4, 2, 4)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    a[1, 777] = 4
    with pytest.raises(ValueError):
        gpu.cp_eval(g, a, w.speeds, w.bandwidth, out_layout=1)
    g.close()


def test_not_where_other_plans_are_faster(gpu, oracle):
    """Wide levels: 300 of 500 vertices and 48 partitions took 330 us in the chain sweep, 268 in the resident-window plan."""
    _check(gpu, oracle, _graph(12, [500] * 300, 5, 6, 48, 16), 1, chain=False)
    _check(gpu, oracle, _graph(12, [500] * 300, 5, 6, 8, 16), 1)
    # and vertex numbers in no relation to the levels: 300 of 400 and 64 partitions, one sweep 608 us, 280 in that plan
    for width, P, chain in ((400, 64, False), (40, 2, True)):
        w = _graph(13, [width] * 300, 7, 4, P, 10)
        name = np.random.default_rng(1).permutation(w.n)
        src, c, level = np.repeat(np.arange(w.n), np.diff(w.succ_ptr)), np.empty(w.n, np.int64), np.empty(w.n, np.int64)
        c[name], level[name] = w.c, w.level
        w = T._custom("scattered", w.n, name[src], name[w.succ_idx], w.succ_t, c, w.speeds, w.bandwidth, w.assignments, level)
        _check(gpu, oracle, w, 1, chain=chain)


@pytest.mark.parametrize("room,rounds", [(1, 7), (2, 4), (3, 3), (4, 2), (6, 2), (7, 1)])
@pytest.mark.parametrize("layout,tick_bytes", [(0, 4), (1, 4), (0, 8), (1, 8)])
def test_in_rounds_where_the_workspace_holds_fewer_partitions(gpu, oracle, layout, tick_bytes, room, rounds):
    import torch
    w = _graph(11, [211] * 260, 7, 10, 7, 16)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    ref = oracle.evaluate_workload(w, threads=8)
    size = binding.workspace_bytes(g, room, w.k, out_layout=layout, tick_bytes=tick_bytes)
    work = torch.empty(size, dtype=torch.uint8, device="cuda:0")
    prof = gpu.CpProfile(1)
    out = gpu.cp_eval(g, a, w.speeds, w.bandwidth, out_layout=layout, tick_bytes=tick_bytes, workspace=work, profile=prof)
    rows = (lambda x: x.cpu().numpy()) if layout == 1 else (lambda x: x.cpu().numpy().T)
    assert np.array_equal(out["cp"].cpu().numpy(), ref["cp"])
    for key in ("b", "tl"):
        assert np.array_equal(rows(out[key]).astype(np.int64), ref[key]), key
    assert prof.plan(0) == gpu.PLAN_CHAIN or rounds > 2       # (three take as long as what other plans do)
    if prof.plan(0) == gpu.PLAN_CHAIN:
        assert prof.read(0)[1] == (rounds, 0)
    g.close()
