"""One partition's path by jumps of eight (cp_search, cp_seed_partition on 128 levels and more): path lengths around
multiples of the jump, rows shared out over the wavefront, ties, every width of weights and ticks, and the walk that
serves a workspace without room for the jumps."""
import ctypes

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


def _seed_equal(gpu, oracle, w):
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    got = gpu.cp_seed_partition(g, w.speeds).cpu().numpy()
    g.close()
    assert np.array_equal(got, oracle.seed(w.n, w.succ_ptr, w.succ_idx, w.c, w.speeds, max_len=w.L))


def _old_size(gpu, oracle, w):
    """The workspace as it was without the jumps: their bytes, three words a vertex and one, taken off again."""
    import torch
    lib = gpu.load_library()
    g = gpu.CpGraph.from_workload(w, device="cuda:0")
    need = ctypes.c_size_t(0)
    assert lib.cp_seed_workspace_bytes(g._handle, ctypes.byref(need)) == 0
    jumps = (12 * (w.n + 1) + 255) // 256 * 256
    s = np.ascontiguousarray(w.speeds, dtype=np.int64)
    ref = oracle.seed(w.n, w.succ_ptr, w.succ_idx, w.c, w.speeds, max_len=w.L)
    for size, answer in ((need.value, True), (need.value - 1, True), (need.value - jumps, True),
                         (need.value - jumps - 1, False)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda:0")
        out = torch.empty(w.n, dtype=torch.uint8, device="cuda:0")
        status = torch.empty(1, dtype=torch.int32, device="cuda:0")
        rc = lib.cp_seed_partition(g._handle, len(s), s.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)),
                                   ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(size), None,
                                   ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(status.data_ptr()))
        torch.cuda.synchronize()
        assert (rc == 0) == answer
        if answer:
            assert np.array_equal(out.cpu().numpy(), ref)
    g.close()


@pytest.mark.parametrize("levels", [127, 128, 129, 135, 136, 137, 255, 257])
def test_lengths_of_a_chain(gpu, oracle, levels):
    rng = np.random.default_rng(levels)
    src, dst = np.arange(levels - 1), np.arange(1, levels)
    w = T._custom("chain", levels, src, dst, rng.integers(0, 50, levels - 1), rng.integers(0, 9, levels), [1, 3],
                  [[1, 2], [5, 1]], rng.integers(0, 2, (1, levels), dtype=np.uint8), np.arange(levels))
    _seed_equal(gpu, oracle, w)
    T._check_search(gpu, oracle, w, w.assignments[0], max_moves=2)


@pytest.mark.parametrize("widths,deg,span,k,c_hi,t_hi", [
    ([3] * 300, 2, 9, 4, 2, 2),                  # ties everywhere, ends on many levels
    ([40, 1] * 70, 36, 3, 4, 50, 200),           # rows of 32 edges and more
    ([5] * 150, 3, 4, 100, 50, 200),
    ([4] * 140, 3, 5, 6, 2 ** 33, 2 ** 40),      # weights past 32 bits
    ([3] * 130, 3, 4, 3, 2 ** 26, 2 ** 28),      # 64-bit ticks from 32-bit weights
])
def test_paths_equal_the_oracles(gpu, oracle, widths, deg, span, k, c_hi, t_hi):
    w = _random(len(widths) + k, widths, deg, span, k, c_hi, t_hi)
    if k <= 64:
        _seed_equal(gpu, oracle, w)
    T._check_search(gpu, oracle, w, w.assignments[0], max_moves=3)


def test_a_workspace_without_room_for_the_jumps(gpu, oracle):
    _old_size(gpu, oracle, _random(5, [6] * 140, 3, 4, 4, 50, 200))
