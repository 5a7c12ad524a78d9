"""Scratch of the 2-wave build's kernels beside the Dormand-Prince ones, from the
compiler's resource report: none for the Runge-Kutta forms of the Kerr metric, at
most a few registers for Bulirsch-Stoer and the q-metric, and for the one kernel
that keeps its constants in registers at the price of scratch no more than it has."""
import re

import pytest

from tests.test_kernel_resources import _resources

pytestmark = pytest.mark.slow


def test_two_wave_build_scratch_of_the_other_schemes(tmp_path):
    res = _resources("kt_trace.hip", [], tmp_path)
    seen = 0
    for name, r in res.items():
        m = re.search(r"trace_kernelILi(\d)ELi(\d)ELb(\d)ELi(\d)E", name)
        method, _, batch, metric = (int(v) for v in m.groups())
        assert r["Occupancy"] >= 2, (name, r)
        if method == 1:
            continue
        seen += 1
        if method == 4 and not batch and metric != 1:
            bound = 116
        elif method in (4, 5) or metric == 1:
            bound = 28
        else:
            bound = 0
        assert r["ScratchSize"] <= bound, (name, r, bound)
    assert seen >= 14
