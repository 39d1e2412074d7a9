"""The search's level ranges around the levels that a workgroup raises by itself: levels of thousands of vertices, and
workgroups that reach past those levels."""
import pytest

import test_gpu_parity as T
from test_gpu_search_moves import _random

pytestmark = pytest.mark.gpu

gpu = T.gpu


@pytest.mark.parametrize("widths,deg,span", [
    ([1500] * 4, 3, 3),                          # all of a workgroup on one level
    ([100, 156, 100] * 5, 4, 14),                # a workgroup begins inside a level
    ([8] * 64, 3, 40),                           # exactly 32 levels a workgroup, edges past them
    ([2] * 150, 3, 100),                         # 128 levels a workgroup
])
def test_levels_in_and_past_a_workgroup(gpu, oracle, widths, deg, span):
    w = _random(len(widths), widths, deg, span, 3, 50, 200)
    T._check_search(gpu, oracle, w, w.assignments[0], max_moves=4)
