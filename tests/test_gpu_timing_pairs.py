"""Timing on the small two-dimensional grids that take two steps per launch: a
timed launch is one step, and the results are the same."""
import numpy as np
import pytest

from paper_1907_13415_amd import inputs
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

PARAMS = (1.0, 2.72, 0.05, 0.3, 0.7, 1.3)


@pytest.mark.parametrize("precision", ["fp64", "fp32sr"])
def test_timed_launches_of_paired_steps(precision):
    require_gpu()
    from paper_1907_13415_amd import lc
    out = []
    for timed in (False, True):
        s = lc.Solver("D2Q9", precision, (1, 41, 53), PARAMS)
        s.load(inputs.random_q5((1, 41, 53), np.random.default_rng(5), amp=0.1))
        s.step(6)
        lc.lc_set_timing(s.ctx, timed)
        s.step(9)
        ms, n = lc.lc_get_timing(s.ctx)
        assert n == ([9, 0] if timed else [0, 0]) and (ms[0] > 0) == timed and ms[1] == 0
        lc.lc_set_timing(s.ctx, False)
        s.step(7)
        out.append((s.export(lc.LC_FIELD_F), s.export(lc.LC_FIELD_Q)))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
