"""The search's candidates are compared without evaluating them one by one: graphs and constraints
where that bookkeeping has edges, move by move against the oracle."""
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


def _random(seed, widths, deg, span, k, c_hi, t_hi, extra=()):
    rng = np.random.default_rng(seed)
    n, level, src, dst = random_layered_dag(rng, widths, 1, deg, span)
    src, dst = (np.concatenate([x, [e[i] for e in extra]]).astype(np.int64) for i, x in enumerate((src, dst)))
    keep = np.ones(len(src), dtype=bool)
    keep[rng.choice(len(src), len(src) // 8, replace=False)] = False      # sources and sinks on every level
    src, dst = src[keep], dst[keep]
    return T._custom("moves", n, src, dst, rng.integers(0, t_hi, len(src)), rng.integers(0, c_hi, n),
                     rng.integers(1, 9, k), rng.integers(1, 20, (k, k)),
                     rng.integers(0, k, (2, n), dtype=np.uint8), level)


@pytest.mark.parametrize("widths,deg,span,k,c_hi,t_hi", [
    ([1] * 3, 1, 1, 2, 9, 9),                    # one vertex a level: nothing avoids it but early sinks and late sources
    ([7] * 40, 3, 30, 5, 50, 200),               # edges over every number of levels
    ([40, 1, 40, 1, 40], 36, 3, 4, 50, 200),     # rows of 32 edges and more, single vertices between
    ([5] * 33, 4, 5, 64, 50, 200),               # as many devices as lanes
    ([6] * 20, 4, 5, 100, 50, 200),              # more devices than lanes
    ([6] * 20, 4, 5, 6, 2 ** 33, 2 ** 40),       # weights past 32 bits
    ([3] * 70, 3, 4, 3, 2 ** 26, 2 ** 28),       # 64-bit ticks from 32-bit weights
])
def test_moves_equal_the_oracles(gpu, oracle, widths, deg, span, k, c_hi, t_hi):
    w = _random(len(widths) + k, widths, deg, span, k, c_hi, t_hi)
    for start in w.assignments:
        got = T._check_search(gpu, oracle, w, start, max_moves=6)
        assert got["evaluated"] % (k - 1) == 0


def test_more_levels_than_one_workgroup_folds(gpu, oracle):
    n = 5001
    w = _random(3, [1] * n, 2, 3, 2, 30, 60, extra=((0, n - 1), (5, 4990), (17, 2100)))
    T._check_search(gpu, oracle, w, w.assignments[0], max_moves=2)


def test_constraints_that_are_broken_at_the_start(gpu, oracle):
    w = _random(9, [6] * 25, 3, 4, 4, 50, 200)
    a = w.assignments[0].astype(int)
    free = T._check_search(gpu, oracle, w, w.assignments[0], max_moves=1)
    v, d = (int(x) for x in free["moves"][0])
    other = next(u for u in range(w.n) if u != v and a[u] == d)
    apart = next(u for u in range(w.n) if u != v and a[u] != d and a[u] != a[v])
    for pairs, pins in (((), [[v, d]]),                        # mended by the best move
                        ([[v, other]], [[v, d], [v, d]]),      # the same asked for more than once
                        ([[v, other], [other, v], [v, v]], ()),
                        ([[v, other], [v, apart]], ()),        # two devices asked for: no move is valid
                        ([[v, other], [other, apart]], ()),    # one that no path vertex can mend
                        ((), [[v, d], [other, (d + 1) % 4]])):
        T._check_search(gpu, oracle, w, w.assignments[0], pairs=pairs, pins=pins, max_moves=3)
