"""What a batch says about the launches of its steps, and that another batch of
the same grids can be made to run them."""
import numpy as np
import pytest

from paper_1907_13415_amd import inputs
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

PARAMS = (1.0, 2.72, 0.05, 0.3, 0.7, 1.3)
LARGE = [(400, 500), (600, 560), (57, 9)]  # 640^2 sites and more: strips by default
SMALL = [(23, 37), (64, 64), (40, 96)]


def _batch(lc, shapes, precision="fp32dev"):
    b = lc.BatchSolver(precision, shapes, [PARAMS] * len(shapes))
    _load(b, shapes)
    return b


def _load(b, shapes):
    for k, s in enumerate(shapes):
        b.load(k, inputs.random_q5((1,) + s, np.random.default_rng(k), amp=0.05))


def _state(lc, b):
    return [b.export(k, f) for k in range(b.n) for f in (lc.LC_FIELD_F, lc.LC_FIELD_Q)]


def test_launch_as_set():
    """Tiles turn the strips off, strips keep the tiles; the same results
    through graphs of every form in turn."""
    require_gpu()
    from paper_1907_13415_amd import lc
    assert _batch(lc, SMALL).launch() == (False, 0, 0)
    a, b = _batch(lc, LARGE), _batch(lc, LARGE)
    assert a.launch() == (True, 0, 0)
    for step, (call, args, launch) in enumerate([("set_tiles", (4, 1), (False, 4, 1)), ("set_strips", (1,), (True, 4, 1)),
                                                 ("set_strips", (0,), (False, 4, 1)), ("set_tiles", (5, 5), (False, 5, 5))]):
        getattr(a, call)(*args)
        assert a.launch() == launch
        a.step(65 + step)
        b.step(65 + step)
    assert all(np.array_equal(x, y) for x, y in zip(_state(lc, a), _state(lc, b)))


@pytest.mark.parametrize("shapes", [LARGE, SMALL])
def test_tuned_launch_carries_over(shapes):
    """The tuner's choice, strips or a pair of tiles, is what the batch says it
    runs, and another batch can be set to it."""
    require_gpu()
    from paper_1907_13415_amd import lc
    print("tuned launch of %s" % (shapes,), flush=True)
    a, b = _batch(lc, shapes), _batch(lc, shapes)
    chosen, ms = a.autotune(3)
    strips, v_lb, v_q = a.launch()
    print("strips %s, tiles %d %d, %.4f ms" % (strips, v_lb, v_q, ms), flush=True)
    assert 0 <= chosen < 49 and (v_lb, v_q) == (chosen % 7, chosen // 7) and ms > 0
    b.set_tiles(v_lb, v_q)
    b.set_strips(strips)
    assert b.launch() == a.launch()
    _load(a, shapes)
    _load(b, shapes)
    a.step(66)
    b.step(66)
    assert all(np.array_equal(x, y) for x, y in zip(_state(lc, a), _state(lc, b)))


@pytest.mark.parametrize("precision,trial", [("fp32sr", 3), ("fp64", 64), ("fp32dev", 70)])
def test_tuning_advances_the_state_by_its_trials(precision, trial):
    """49 times (trial + 1) steps, also with trials that replay graphs, and none
    for the strips: the state is that of as many plain steps."""
    require_gpu()
    from paper_1907_13415_amd import lc
    print("tuning state %s %d" % (precision, trial), flush=True)
    a, b = _batch(lc, SMALL, precision), _batch(lc, SMALL, precision)
    a.autotune(trial)
    b.step(49 * (trial + 1))
    assert a.observe()[0]["step"] == 49 * (trial + 1)
    assert all(np.array_equal(x, y) for x, y in zip(_state(lc, a), _state(lc, b)))
    a.step(67)
    b.step(67)
    assert all(np.array_equal(x, y) for x, y in zip(_state(lc, a), _state(lc, b)))
