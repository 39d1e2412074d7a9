"""What cp_eval's workspace grows by for the sweep of a few partitions of a deep graph (CP_PLAN_CHAIN).  No kernel is launched."""
import functools

import numpy as np
import pytest

from paper_1711_01912_amd import CpGraph, OUT_PARTITION_MAJOR, OUT_VERTEX_MAJOR, binding
from workloads import build_csr

MOST = 512 << 20
TABLES = 1 << 16         # of 16 devices, and alignment


@functools.lru_cache(maxsize=None)
def _graph(levels, width, max_t, degree=2):
    n = levels * width
    rng = np.random.default_rng(1)
    src = np.repeat(np.arange(n - width), degree)
    dst = (src // width + 1) * width + rng.integers(0, width, len(src))
    csr = build_csr(n, src, dst, rng.integers(max_t // 2, max_t + 1, len(src)), np.arange(n) // width)
    c = rng.integers(1, 100, n)
    c[0] = 100
    names = ("succ_ptr", "succ_idx", "succ_t", "pred_ptr", "pred_idx", "pred_eid", "level_ptr", "level_vtx")
    return CpGraph(n=n, c=c, **{name: csr[name] for name in names})


def _bytes(g, batch, layout, tick=4):
    return binding.workspace_bytes(g, batch, 16, out_layout=layout, tick_bytes=tick)


@pytest.mark.parametrize("layout", [OUT_VERTEX_MAJOR, OUT_PARTITION_MAJOR])
def test_a_million_vertices(layout):
    g = _graph(2000, 500, 10_000)
    few = [_bytes(g, batch, layout) for batch in (1, 8, 16, 32, 64)]
    assert few == sorted(few)
    assert few[-1] <= _bytes(g, 256, layout)
    assert few[-1] <= max(MOST + TABLES, _bytes(g, 65, layout))


def test_costs_that_fit_16_bits_take_half():
    small, large = _graph(300, 60, 60_000), _graph(300, 60, 70_000)
    for batch in (1, 17, 64):
        half, whole = (_bytes(g, batch, OUT_VERTEX_MAJOR) for g in (small, large))
        assert half < 0.55 * whole


def test_rows_that_the_sweep_cannot_write():
    """Rows per vertex of 64-bit ticks: past 32 partitions another plan runs, and nothing is asked for."""
    g = _graph(300, 60, 60_000)
    assert _bytes(g, 33, OUT_VERTEX_MAJOR, 8) < _bytes(g, 32, OUT_VERTEX_MAJOR, 8)
    assert _bytes(g, 33, OUT_VERTEX_MAJOR, 8) <= _bytes(g, 65, OUT_VERTEX_MAJOR, 8)
