"""The benchmark names every plan that a call can run."""
import os
import sys

import paper_1711_01912_amd as cpe

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


def test_every_plan_has_a_name():
    import bench
    plans = {getattr(cpe, name) for name in dir(cpe) if name.startswith("PLAN_")} - {cpe.PLAN_AUTO}
    assert plans == set(bench.PLAN_NAMES)
