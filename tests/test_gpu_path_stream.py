"""Walks over records with b and the device ids streamed through a ring of LDS (rows along partitions, edges to later vertices
only): rings that go round several times, both sizes, a reach just within and past them, starts far from vertex 0, edges that
skip whole chunks, vertices in no order, rows longer than a record, device ids that are too large."""
import numpy as np
import pytest

import test_gpu_parity as T
from test_gpu_path_records import _check, gpu  # noqa: F401
from workloads import random_layered_dag

pytestmark = pytest.mark.gpu


def _graph(seed, widths, deg, span, P, k, order=None, lone=0):
    rng = np.random.default_rng(seed)
    n, level, src, dst = random_layered_dag(rng, widths, 1, deg, span)
    if lone:                                     # vertices without edges in front of the others
        src, dst, level, n = src + lone, dst + lone, np.concatenate([np.zeros(lone, dtype=level.dtype), level]), n + lone
    if order is not None:
        name = rng.permutation(n)
        src, dst, old = name[src], name[dst], level
        level = np.empty_like(old)
        level[name] = old
    return T._custom("stream", n, src, dst, rng.integers(0, 300, len(src)), rng.integers(0, 50, n), rng.integers(1, 9, k),
                     rng.integers(1, 20, (k, k)), rng.integers(0, k, (P, n), dtype=np.uint8), level)


@pytest.mark.parametrize("kw", [
    dict(widths=[100] * 300, deg=5, span=5, P=64, k=4),          # the ring goes round seven times
    dict(widths=[260] * 260, deg=4, span=20, P=64, k=16),        # reach near 5,500: the larger ring
    dict(widths=[61] * 300, deg=3, span=31, P=65, k=2),          # reach near 2,000
    dict(widths=[400] * 256, deg=3, span=16, P=64, k=3),         # past 6,144: no ring
    dict(widths=[3] * 400, deg=3, span=4, P=1024, k=50),         # less than a chunk for every loader
    dict(widths=[1, 2000] + [1] * 300, deg=2, span=1, P=64, k=3),    # a chunk or more between two vertices
    dict(widths=[20] * 300, deg=5, span=3, P=70, k=5, lone=5000),    # the path begins far behind vertex 0
    dict(widths=[20] * 300, deg=5, span=3, P=70, k=5, order=1),
])
def test_against_the_oracle(gpu, oracle, kw):  # noqa: F811
    _check(gpu, oracle, _graph(11, **kw))


def test_no_start(gpu):  # noqa: F811
    """A cp that no source has: every path is empty and the loaders leave."""
    import torch
    w = _graph(3, [30] * 300, 3, 3, 64, 3)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    out = gpu.cp_eval(g, a, w.speeds, w.bandwidth, want=("cp", "b"), out_layout=1)
    cp = out["cp"] + 1
    cp[2] -= 1
    paths, lens = gpu.cp_critical_path(g, a, w.speeds, w.bandwidth, out["b"], cp, b_layout=1)
    assert lens.cpu().tolist()[:2] == [0, 0] and int(lens[2]) > 0 and bool((paths[0] == -1).all())
    g.close()


@pytest.mark.parametrize("rich", [(7, 9), (8, 12), (60, 70)])
def test_rows_longer_than_a_record(gpu, oracle, rich):  # noqa: F811
    """Four vertices in a level of 40 or 70 with that many out-edges, half of which lead to such vertices of the next level."""
    rng = np.random.default_rng(rich[0])
    levels, width, P = 300, 40 if rich[1] < 20 else 70, 64
    n = levels * width
    deg = np.where(np.arange(n) % width < 4, rng.integers(rich[0], rich[1] + 1, n), rng.integers(0, 2, n))
    deg[n - width:] = 0
    src = np.repeat(np.arange(n), deg)
    to = (src // width + 1) * width
    dst = to + np.where(rng.random(len(src)) < 0.5, rng.integers(0, 4, len(src)), rng.integers(0, width, len(src)))
    w = T._custom("rich", n, src, dst, rng.integers(0, 40, len(src)), rng.integers(0, 30, n), [1, 2, 3],
                  rng.integers(1, 5, (3, 3)), rng.integers(0, 3, (P, n), dtype=np.uint8), np.arange(n) // width)
    degree = np.diff(w.succ_ptr)
    assert len(src) // n <= 5 and degree.max() > 7
    lengths = _check(gpu, oracle, w)
    assert lengths.max() > 200                   # (paths go through the long rows: other vertices have one out-edge at most)


@pytest.mark.parametrize("where", [0, 1, 2, 64, 150])
def test_a_device_id_too_large_is_reported(gpu, where):  # noqa: F811
    import torch
    w = _graph(5, [30] * 300, 3, 3, 64, 3)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    out = gpu.cp_eval(g, a, w.speeds, w.bandwidth, want=("cp", "b"), out_layout=1)
    paths, lens = gpu.cp_critical_path(g, a, w.speeds, w.bandwidth, out["b"], out["cp"], b_layout=1)
    for q in (0, 63):
        # a vertex of the last device, which a larger id counts as where it is a candidate: the walk still comes by
        path = paths[q, :int(lens[q])].long()
        v = int(path[where:][a[q, path[where:]] == 2][0])
        a[q, v] = 3
        with pytest.raises(ValueError):
            gpu.cp_critical_path(g, a, w.speeds, w.bandwidth, out["b"], out["cp"], b_layout=1)
        a[q, v] = 2
    again, _ = gpu.cp_critical_path(g, a, w.speeds, w.bandwidth, out["b"], out["cp"], b_layout=1)
    assert bool((again == paths).all())
    g.close()
