"""cp_critical_path's two walks, over records (256 levels and more, five edges a vertex at most, room in the workspace) and
over the CSR: path lengths
around the 64 vertices that are stored together, out-degrees around the seven edges of a record, both tick widths and
layouts, weights without multiply-shift constants."""
import numpy as np
import pytest

from workloads import random_layered_dag

import test_gpu_parity as T
from test_gpu_search_moves import _random

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1711_01912_amd as cpe
    cpe.load_library()
    return cpe


def _check(gpu, oracle, w):
    import torch
    from paper_1711_01912_amd import binding
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    ref_p, ref_l = oracle.critical_path(w.n, w.succ_ptr, w.succ_idx, w.succ_t, w.c, w.speeds, w.bandwidth,
                                        w.assignments, max_len=w.L)
    k = len(w.speeds)
    tables = ((2 * k * k + 2 * k) * 8 + (2 * k * k + 2 * k) * 4 + 4096) // 256 * 256      # at least the tables' bytes
    enough = max(binding.workspace_bytes(g, w.P, k), tables + 64 * w.n + 256)
    for layout in (0, 1):
        a = torch.from_numpy(w.assignments if layout == 0 else np.ascontiguousarray(w.assignments.T)).to("cuda:0")
        for ol in (0, 1):
            out = gpu.cp_eval(g, a, w.speeds, w.bandwidth, want=("cp", "b"), assign_layout=layout, out_layout=ol)
            for size in (enough, tables):        # with room for the records and without
                ws = torch.empty(size, dtype=torch.uint8, device="cuda:0")
                paths, lens = gpu.cp_critical_path(g, a, w.speeds, w.bandwidth, out["b"], out["cp"],
                                                   assign_layout=layout, b_layout=ol, workspace=ws)
                assert np.array_equal(lens.cpu().numpy(), ref_l)
                assert np.array_equal(paths.cpu().numpy(), ref_p)
    g.close()
    return ref_l


@pytest.mark.parametrize("levels", [1, 63, 64, 65, 128, 255, 256, 257, 319, 320, 321])
def test_lengths_of_a_chain(gpu, oracle, levels):
    rng = np.random.default_rng(levels)
    src, dst = np.arange(levels - 1), np.arange(1, levels)
    w = T._custom("chain", levels, src, dst, rng.integers(0, 50, levels - 1), rng.integers(0, 9, levels), [1, 3],
                  [[1, 2], [5, 1]], rng.integers(0, 2, (5, levels), dtype=np.uint8), np.arange(levels))
    assert np.all(_check(gpu, oracle, w) == levels)


@pytest.mark.parametrize("degree", [1, 4, 5, 7, 8, 9, 65])
def test_degrees(gpu, oracle, degree):
    # every second level one vertex with exactly this many successors
    rng = np.random.default_rng(degree)
    levels, width = 260, degree + 1
    at = np.arange(levels // 2 - 1)
    hub, fan = 2 * at * width, (2 * at + 1) * width
    src = np.concatenate([np.repeat(hub, degree), (fan[:, None] + np.arange(degree)).ravel()])
    dst = np.concatenate([(fan[:, None] + np.arange(degree)).ravel(), np.repeat(hub + 2 * width, degree)])
    order = np.argsort(src, kind="stable")
    n = levels * width
    level = np.zeros(n, dtype=np.int64)
    level[hub], level[(fan[:, None] + np.arange(degree)).ravel()] = 2 * at, np.repeat(2 * at + 1, degree)
    level[2 * len(at) * width] = 2 * len(at)
    w = T._custom("degrees", n, src[order], dst[order], rng.integers(0, 4, len(src)), rng.integers(0, 3, n), [1, 2, 5],
                  rng.integers(1, 4, (3, 3)), rng.integers(0, 3, (7, n), dtype=np.uint8), level)
    _check(gpu, oracle, w)


@pytest.mark.parametrize("rich", [(8, 12), (7, 9), (60, 70), (1, 100)])
def test_long_rows_after_each_other(gpu, oracle, rich):
    """Paths through rows of more than a record's seven edges: one after the other, before and after short rows."""
    rng = np.random.default_rng(rich[0])
    levels, width = 270, 120
    n = levels * width
    deg = np.where(np.arange(n) % width < 4, rng.integers(rich[0], rich[1] + 1, n), rng.integers(0, 3, n))
    deg[-width:] = 0
    src = np.repeat(np.arange(n), deg)
    # half of the edges go to the four rich vertices of the next level
    dst = (src // width + 1) * width + np.where(rng.random(len(src)) < 0.5, rng.integers(0, 4, len(src)),
                                                rng.integers(0, width, len(src)))
    w = T._custom("rich", n, src, dst, rng.integers(0, 40, len(src)), rng.integers(0, 30, n), [1, 2, 3],
                  rng.integers(1, 4, (3, 3)), rng.integers(0, 3, (9, n), dtype=np.uint8), np.arange(n) // width)
    assert len(src) <= 5 * n
    _check(gpu, oracle, w)


@pytest.mark.parametrize("widths,deg,span,k,c_hi,t_hi", [
    ([4] * 300, 2, 9, 4, 2, 2),                  # ties everywhere, ends on many levels
    ([9] * 270, 12, 4, 64, 50, 200),             # rows of up to twelve edges, as many devices as LDS tables take
    ([5] * 260, 3, 4, 65, 50, 200),              # one more
    ([4] * 260, 3, 5, 6, 2 ** 33, 2 ** 40),      # weights past 32 bits
    ([3] * 260, 3, 4, 3, 2 ** 26, 2 ** 28),      # 64-bit ticks from 32-bit weights
])
def test_paths_equal_the_oracles(gpu, oracle, widths, deg, span, k, c_hi, t_hi):
    _check(gpu, oracle, _random(len(widths) + k, widths, deg, span, k, c_hi, t_hi))


@pytest.mark.parametrize("room", [True, False])
@pytest.mark.parametrize("where", [0, 100, 299])
def test_a_device_id_too_large_is_reported(gpu, where, room):
    """On the path of a chain, over records and over the CSR: reported, and the call returns.  All vertices are on the last
    device, whose costs a larger id is given, so that the path reaches it."""
    import torch
    n, k = 300, 3
    src, dst = np.arange(n - 1), np.arange(1, n)
    w = T._custom("bad-id", n, src, dst, np.full(n - 1, 5), np.full(n, 2), [1] * k, np.ones((k, k), dtype=np.int64),
                  np.full((2, n), k - 1, dtype=np.uint8), np.arange(n))
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    a = torch.from_numpy(w.assignments).to("cuda:0")
    out = gpu.cp_eval(g, a, w.speeds, w.bandwidth, want=("cp", "b"), out_layout=1)
    ws = torch.empty(4096 + (64 * n if room else 0), dtype=torch.uint8, device="cuda:0")
    paths, lens = gpu.cp_critical_path(g, a, w.speeds, w.bandwidth, out["b"], out["cp"], b_layout=1, workspace=ws)
    assert lens.tolist() == [n, n]
    a[1, where] = k
    with pytest.raises(ValueError):
        gpu.cp_critical_path(g, a, w.speeds, w.bandwidth, out["b"], out["cp"], b_layout=1, workspace=ws)
    g.close()
