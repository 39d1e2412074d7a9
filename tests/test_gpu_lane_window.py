"""The lane-window plan against the oracle at the edges of its packets, its groups of lanes and its ring."""
import numpy as np
import pytest

from workloads import make_workload, random_layered_dag

import test_gpu_parity as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1711_01912_amd as cpe
    cpe.load_library()
    return cpe


def _case(seed, widths, deg, span, k, P, c_hi=50, t_hi=300, rates=20, extra=0, renumber=False):
    rng = np.random.default_rng(seed)
    n, level, src, dst = random_layered_dag(rng, widths, 1, deg, span)
    if extra:                                     # rows of several sub-rows: one vertex feeds and one reads a whole level
        first, last = np.arange(widths[0]), np.arange(n - widths[-1], n)
        src = np.concatenate([src, np.zeros(len(last), dtype=np.int64), first[1:]])
        dst = np.concatenate([dst, last, np.full(len(first) - 1, n - 1)])
    if renumber:
        name = rng.permutation(n)
        old, level = level, np.empty_like(level)
        level[name] = old
        src, dst = name[src], name[dst]
    return T._custom("lanes", n, src, dst, rng.integers(0, t_hi, len(src)), rng.integers(0, c_hi, n),
                     rng.integers(1, 9, k), rng.integers(1, rates, (k, k)), rng.integers(0, k, (P, n), dtype=np.uint8),
                     level)


def _check(gpu, oracle, w, **kw):
    from gpu_util import assert_equal_to_oracle, run_gpu
    ref = oracle.evaluate_workload(w, threads=8)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    for layout, out_layout in ((0, 1), (1, 0), (0, 0)):
        res = run_gpu(w, gpu.PLAN_LANE_WINDOW, layout=layout, graph=g, out_layout=out_layout, **kw)
        assert_equal_to_oracle(res, ref, f"layout {layout}, outputs {out_layout}")
    for want in (("cp",), ("tl",), ("b",)):       # one sweep alone
        res = run_gpu(w, gpu.PLAN_LANE_WINDOW, graph=g, out_layout=1, want=want, **kw)
        assert set(res) == set(want)              # CP alone writes no b, with far reads neither
        for key in want:
            assert np.array_equal(res[key], ref[key]), key
    g.close()


@pytest.mark.parametrize("P", [1, 7, 8, 9, 33, 300, 3000])
def test_batches_around_a_group(gpu, oracle, P):
    _check(gpu, oracle, _case(P, [9] * 12, 3, 3, 5, P))


@pytest.mark.parametrize("widths,deg,span,extra", [
    ([1], 1, 1, 0), ([1] * 9, 2, 3, 0), ([3, 70, 1, 64, 65, 2], 9, 2, 0),
    ([300, 1, 520, 255, 256, 257], 3, 1, 0),      # levels cut into ticks, ticks of one vertex between
    ([40] * 6, 8, 5, 1), ([17] * 30, 17, 4, 1),   # sub-rows of every length, vertices of many sub-rows
])
def test_levels_and_rows(gpu, oracle, widths, deg, span, extra):
    for renumber in (False, True):
        _check(gpu, oracle, _case(len(widths) + deg, widths, deg, span, 4, 37, extra=extra, renumber=renumber))


@pytest.mark.parametrize("k", [1, 2, 33, 64])
def test_device_counts(gpu, oracle, k):
    _check(gpu, oracle, _case(k, [11] * 9, 4, 3, k, 41))


@pytest.mark.parametrize("c_hi,t_hi,rates", [(2 ** 20, 2 ** 28, 64), (2 ** 31, 2 ** 31, 3), (9, 2 ** 31, 2 ** 20)])
def test_weights_that_need_the_remainder(gpu, oracle, c_hi, t_hi, rates):
    w = _case(5, [13] * 40, 4, 4, 6, 50, c_hi=c_hi, t_hi=t_hi, rates=rates)
    _check(gpu, oracle, w)


def test_64_bit_ticks_of_a_small_graph_and_the_perceptron(gpu, oracle):
    _check(gpu, oracle, _case(8, [9] * 12, 3, 3, 5, 20), tick_bytes=8)
    _check(gpu, oracle, make_workload("mlp", P=70))


@pytest.mark.parametrize("widths,P,far", [([30] * 120, 37, "all"), ([50, 3] * 60, 9, "all"), ([30] * 120, 8, "few")])
def test_neighbours_too_far_back_for_the_ring(gpu, oracle, widths, P, far):
    """Every vertex of the first half also feeds its mirror image in the second half; the ring holds neither sweep."""
    rng = np.random.default_rng(len(widths) + P)
    n, level, src, dst = random_layered_dag(rng, widths, 1, 3, 2)
    x = np.arange(n // 2)
    if far == "few":                              # a long edge here and there, ticks without any between
        x = x[::97]
    x = x[level[n - 1 - x] > level[x]]
    src, dst = np.concatenate([src, x]), np.concatenate([dst, n - 1 - x])
    w = T._custom("far", n, src, dst, rng.integers(0, 300, len(src)), rng.integers(0, 50, n), rng.integers(1, 9, 5),
                  rng.integers(1, 20, (5, 5)), rng.integers(0, 5, (P, n), dtype=np.uint8), level)
    _check(gpu, oracle, w)


def test_far_reads_of_the_modules_and_with_64_bit_words(gpu, oracle):
    _check(gpu, oracle, make_workload("inception", P=11))
    w = make_workload("inception", P=9, modules=12)
    w.succ_t[:] = w.succ_t * 1000
    _check(gpu, oracle, w)


def test_bad_device_id_and_refusals(gpu):
    import torch
    w = _case(3, [9] * 12, 3, 3, 5, 20)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments.copy()).to("cuda:0")
    a[19, w.n - 1] = 5
    with pytest.raises(ValueError):
        gpu.cp_eval(g, a, w.speeds, w.bandwidth, plan=gpu.PLAN_LANE_WINDOW)
    wide = _case(4, [3000] * 4, 2, 1, 3, 2)       # the ring of the smallest group does not fit
    g2 = gpu.CpGraph.from_workload(wide, device="cuda:0")
    with pytest.raises(gpu.CpError) as e:
        gpu.cp_eval(g2, torch.from_numpy(wide.assignments).to("cuda:0"), wide.speeds, wide.bandwidth,
                    plan=gpu.PLAN_LANE_WINDOW)
    assert e.value.code == -12
    g.close()
    g2.close()


def test_batches_past_the_grid(gpu, oracle):
    """More groups of eight than a grid's second dimension takes: refused by name, still evaluated under AUTO."""
    w = _case(6, [2] * 4, 2, 2, 3, 8 * 65535 + 1)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    import torch
    a = torch.from_numpy(w.assignments).to("cuda:0")
    with pytest.raises(gpu.CpError) as e:
        gpu.cp_eval(g, a, w.speeds, w.bandwidth, plan=gpu.PLAN_LANE_WINDOW)
    assert e.value.code == -12
    from gpu_util import assert_equal_to_oracle, run_gpu
    assert_equal_to_oracle(run_gpu(w, gpu.PLAN_AUTO, graph=g, out_layout=1), oracle.evaluate_workload(w, threads=8), "auto")
    g.close()


@pytest.mark.parametrize("P", [3, 300])
@pytest.mark.parametrize("which", ["far", "column"])
def test_cp_without_b_stays_refused_under_auto(gpu, oracle, which, P, monkeypatch):
    """Where the plan beside the lanes needs b for CP, AUTO refuses CP alone whatever it would take; the binding adds b."""
    from gpu_util import run_gpu
    w = make_workload("inception", P=P) if which == "far" else _case(7, [9] * 12, 3, 3, 5, P, t_hi=2 ** 31)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    ref = oracle.evaluate_workload(w, threads=8)["cp"]
    assert np.array_equal(run_gpu(w, gpu.PLAN_AUTO, want=("cp",), graph=g)["cp"], ref)
    from paper_1711_01912_amd import binding
    info = dict(g.info, window_far_b=0)
    monkeypatch.setattr(binding.CpGraph, "info", property(lambda self: info))
    monkeypatch.setattr(binding, "choose_plan", lambda *a: gpu.PLAN_RESIDENT_WINDOW)
    with pytest.raises(gpu.CpError) as e:
        run_gpu(w, gpu.PLAN_AUTO, want=("cp",), graph=g)
    assert e.value.code == -12
    g.close()
