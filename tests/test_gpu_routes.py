"""Grids whose launch rule (tests/test_launch_rules.py) chooses a shape that the
other tests of that kernel do not reach, against the two sweeps bit for bit."""
import numpy as np
import pytest

from paper_1907_13415_amd import inputs
from gpu_util import require_gpu
from test_gpu_vjp_tiles import test_reverse_step_at_tile_edges as reverse_step

pytestmark = pytest.mark.gpu

PARAMS = (1.0, 2.72, 0.05, 0.3, 0.7, 1.3)


def _equal_to_two_sweeps(nx, ny, precision, iso):
    require_gpu()
    from paper_1907_13415_amd import lc
    print("single pass %dx%d %s iso %d" % (nx, ny, precision, iso), flush=True)
    q5 = inputs.random_q5((1, ny, nx), np.random.default_rng(nx + ny), amp=0.1)
    out = []
    for variant in (lc.LC_VARIANT_FUSED, lc.LC_VARIANT_SPLIT):
        s = lc.Solver("D2Q9", precision, (1, ny, nx), PARAMS)
        s.set_variant(variant)
        if iso:
            s.set_stencil(lc.LC_STENCIL_ISOTROPIC)
        s.load(q5)
        s.step(3)
        out.append((s.export(lc.LC_FIELD_F), s.export(lc.LC_FIELD_Q)))
    assert np.isfinite(out[0][1]).all()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("precision,iso", [("fp64", 0), ("fp32sr", 0), ("fp32dev", 1), ("mixed", 0)])
@pytest.mark.parametrize("nx,ny", [(9000, 7), (70, 2000), (449, 447)])
def test_more_tiles_than_compute_units(nx, ny, precision, iso):
    """Two rounds of tiles of 32x8, 32x12 and 32x16 sites."""
    _equal_to_two_sweeps(nx, ny, precision, iso)


# against autograd of the CPU twin, to the bounds of the other tile shape's test
@pytest.mark.parametrize("nx,ny,steps", [(4097, 3, 1), (4120, 4, 2), (5119, 8, 1), (10300, 1, 1)])
def test_reverse_step_in_flat_tiles(nx, ny, steps):
    """40x4 tiles: one short row of tiles, whole tiles, two rows of tiles, a
    single row of sites; last tiles narrower and of whole width."""
    reverse_step(nx, ny, steps)
