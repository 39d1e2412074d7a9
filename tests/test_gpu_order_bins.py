"""Priority lists by bins: spread keys, keys that repeat just under and over what bins take, a partition's keys
crowded among others that are not, buckets of more items than the bins kernel holds, key widths at both ends, and the
sizes where the workgroup changes."""
import numpy as np
import pytest

from workloads import random_layered_dag

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


def _levels(rng, kind, P, n, top):
    b = rng.integers(0, top + 1, (P, n))
    if kind == "mixed":               # the first partitions spread, the others with fewer and fewer values
        for q in range(P):
            b[q] = rng.integers(0, max(2, 20000 >> 2 * q), n) * max(1, top // 20000)
    elif kind == "clusters":          # a third of the vertices within 200 ticks of one value: full buckets and bins
        b[:, : n // 3] = top // 2 + rng.integers(0, 200, (P, n // 3))
    elif kind == "narrow":            # the upper sixteenth of the range only: buckets of several thousand items
        b = top - b // 16
    elif kind == "equal":
        b[:] = top
    return b


@pytest.mark.parametrize("n", [1, 255, 257, 4096, 4097, 16385, 20480, 65536, 70001, 262143, 262145, 524800])
@pytest.mark.parametrize("kind,k,top", [("spread", 16, 2 ** 21 - 1), ("mixed", 7, 1_500_000), ("clusters", 3, 2 ** 30 - 1),
                                        ("narrow", 2, 2 ** 20), ("equal", 50, 2 ** 26 - 1)])
def test_lists_by_bins(gpu, oracle, n, kind, k, top):
    import torch
    rng = np.random.default_rng(n + k)
    P = 9 if n < 100_000 else 3
    if n < 8:
        widths = [n]
    else:
        widths = [n // 2, n - n // 2]
    n, level, src, dst = random_layered_dag(rng, widths, 0 if n < 8 else 1, 1, 1)
    w = T._custom("bins", n, src, dst, np.ones(len(src), dtype=np.int64), np.ones(n, dtype=np.int64), [1] * k,
                  np.ones((k, k), dtype=np.int64), rng.integers(0, k, (P, n), dtype=np.uint8), level)
    b = _levels(rng, kind, P, n, top)
    ref_order, ref_seg = oracle.pct_order(k, w.assignments, b.astype(np.int64), threads=8)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    for layout in (0, 1):
        d = torch.from_numpy(np.ascontiguousarray((b.T if layout == 0 else b).astype(np.int32))).to("cuda:0")
        order, seg = gpu.cp_pct_order(g, a, k, d, max_b=top, b_layout=layout)
        assert np.array_equal(seg.cpu().numpy(), ref_seg)
        assert np.array_equal(order.cpu().numpy(), ref_order)
    g.close()


@pytest.mark.parametrize("n,P", [(65_537, 17), (65_537, 32), (65_537, 65), (65_537, 128), (65_537, 257), (262_145, 17),
                                 (524_801, 20), (65_537, 24), (65_537, 25), (524_801, 48), (524_801, 49)])
def test_left_buckets_among_others(gpu, oracle, n, P):
    """One to sixteen buckets per workgroup of the ranking, one to four of the bins, which have 128, 256 or 512 threads, and
    both in one launch: crowded partitions between spread ones, empty digits (9 of 16 devices) and, in one partition, full
    buckets beside nearly empty ones."""
    import torch
    k, top = 9, 3_000_000
    rng = np.random.default_rng(P)
    n, level, src, dst = random_layered_dag(rng, [n // 2, n - n // 2], 1, 1, 1)
    w = T._custom("left", n, src, dst, np.ones(len(src), dtype=np.int64), np.ones(n, dtype=np.int64), [1] * k,
                  np.ones((k, k), dtype=np.int64), rng.integers(0, k, (P, n), dtype=np.uint8), level)
    b = rng.integers(0, top + 1, (P, n), dtype=np.int32)
    b[::3] = b[::3] // 150_000 * 150_000                     # 21 values
    b[1] = np.where(rng.random(n) < 0.4, top // 2 + b[1] // 1000, b[1])
    ref_order, ref_seg = oracle.pct_order(k, w.assignments, b.astype(np.int64), threads=8)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    order, seg = gpu.cp_pct_order(g, torch.from_numpy(w.assignments).to("cuda:0"), k, torch.from_numpy(b).to("cuda:0"),
                                  max_b=top, b_layout=1)
    assert np.array_equal(seg.cpu().numpy(), ref_seg)
    assert np.array_equal(order.cpu().numpy(), ref_order)
    g.close()


@pytest.mark.parametrize("n,P", [(65_537, 3), (65_537, 65), (262_145, 5), (262_145, 49), (524_801, 5), (524_801, 49)])
def test_a_crowded_bin_among_spread_keys(gpu, oracle, n, P):
    """Too few equal values for the sample to find, too many for a bin: the bucket's items are dealt in no order of their vertex
    numbers and then ranked, in one launch with the bins and in one of its own."""
    import torch
    k, top = 9, 3_000_000
    rng = np.random.default_rng(n + P)
    n, level, src, dst = random_layered_dag(rng, [n // 2, n - n // 2], 1, 1, 1)
    a = rng.integers(0, k, (P, n), dtype=np.uint8)
    w = T._custom("crowded", n, src, dst, np.ones(len(src), dtype=np.int64), np.ones(n, dtype=np.int64), [1] * k,
                  np.ones((k, k), dtype=np.int64), a, level)
    b = rng.integers(0, top + 1, (P, n), dtype=np.int32)
    for q in range(P):
        for d in range(q % 3):
            same = rng.choice(np.nonzero(a[q] == d)[0], 200 + 20 * d, replace=False)
            b[q, same] = top // (d + 2)
    ref_order, ref_seg = oracle.pct_order(k, w.assignments, b.astype(np.int64), threads=8)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    order, seg = gpu.cp_pct_order(g, torch.from_numpy(w.assignments).to("cuda:0"), k, torch.from_numpy(b).to("cuda:0"),
                                  max_b=top, b_layout=1)
    assert np.array_equal(seg.cpu().numpy(), ref_seg)
    assert np.array_equal(order.cpu().numpy(), ref_order)
    g.close()


@pytest.mark.parametrize("n,P", [(65_537, 3), (65_537, 65), (262_145, 5), (262_145, 49), (524_801, 5), (524_801, 49)])
@pytest.mark.parametrize("values", [1, 2, 5])
def test_neighbours_in_a_crowded_bin(gpu, oracle, n, P, values):
    """The same with vertices next to each other, so that all of a wavefront's may be dealt to one bucket: a level of a device's
    vertices with few different values, at the first vertex, at the last one and in between."""
    import torch
    k, top = 9, 3_000_000
    rng = np.random.default_rng([n, P, values])
    n, level, src, dst = random_layered_dag(rng, [n // 2, n - n // 2], 1, 1, 1)
    a = rng.integers(0, k, (P, n), dtype=np.uint8)
    b = rng.integers(0, top + 1, (P, n), dtype=np.int32)
    for q in range(P):
        at, size = [0, n - 300, 1000 + 61 * q, 777][q % 4], 300 if q % 4 < 3 else 150
        a[q, at:at + size] = np.where(rng.random(size) < (1.0 if q % 2 else 0.7), q % k, a[q, at:at + size])
        b[q, at:at + size] = top // 2 - rng.integers(0, values, size)
    w = T._custom("neighbours", n, src, dst, np.ones(len(src), dtype=np.int64), np.ones(n, dtype=np.int64), [1] * k,
                  np.ones((k, k), dtype=np.int64), a, level)
    ref_order, ref_seg = oracle.pct_order(k, w.assignments, b.astype(np.int64), threads=8)
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    order, seg = gpu.cp_pct_order(g, torch.from_numpy(w.assignments).to("cuda:0"), k, torch.from_numpy(b).to("cuda:0"),
                                  max_b=top, b_layout=1)
    assert np.array_equal(seg.cpu().numpy(), ref_seg)
    assert np.array_equal(order.cpu().numpy(), ref_order)
    g.close()
