"""The single pass on two-dimensional grids takes its tile shape from the
number of tiles, and marches along y in strips of 56 columns on large grids:
grids on either side of each change of shape (16x8, 32x8, 32x12, 32x16, 32x20
sites, more tiles than CUs, strips), with and without whole tiles, strips and
chunks of rows, must equal the two sweeps bit for bit in every form."""
import numpy as np
import pytest

from paper_1907_13415_amd import inputs
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

PARAMS = (1.0, 2.72, 0.05, 0.3, 0.7, 1.3)
RATES = (1.64, 1.54, 1.9)
# (nx, ny): 256 and 257 tiles of each shape (nx, ny whole tiles, then ragged)
SHAPES = [(1, 1), (7, 130), (24, 8), (100, 100), (256, 128), (257, 129), (256, 256), (257, 249), (256, 384),
          (225, 385), (256, 512), (259, 513), (256, 640), (301, 419), (300, 641), (5, 9), (39, 27),
          # strips: the smallest grid, whole strips, a last strip of one column, few rows, one chunk of few rows
          (640, 640), (672, 613), (617, 701), (2000, 205), (65000, 7), (65000, 9)]


@pytest.mark.parametrize("nx,ny", SHAPES)
@pytest.mark.parametrize("precision,mrt,iso", [("fp64", False, False), ("fp32dev", True, False),
                                               ("fp32sr", False, False), ("mixed", False, False),
                                               ("fp64", True, True), ("fp32dev", False, True)])
def test_shape_equals_two_sweeps(nx, ny, precision, mrt, iso):
    require_gpu()
    from paper_1907_13415_amd import lc
    print("fused 2D %dx%d %s mrt %d iso %d" % (nx, ny, precision, mrt, iso), flush=True)
    rng = np.random.default_rng(nx + ny)
    q5 = inputs.random_q5((1, ny, nx), rng, amp=0.1)
    f0 = np.array(lc.lc_lattice_info(lc.LC_D2Q9)[1])[:, None, None, None] * (
        1 + inputs.random_rel(9, (1, ny, nx), rng, amp=2e-3))
    out = []
    for variant in (lc.LC_VARIANT_FUSED, lc.LC_VARIANT_SPLIT):
        s = lc.Solver("D2Q9", precision, (1, ny, nx), PARAMS)
        s.set_variant(variant)
        if mrt:
            s.set_collision(lc.LC_COLL_MRT, RATES)
        if iso:
            s.set_stencil(lc.LC_STENCIL_ISOTROPIC)
        s.load(q5, f0)
        s.step(7)  # on the smallest shape two launches of two steps and three of one
        out.append((s.export(lc.LC_FIELD_F), s.export(lc.LC_FIELD_Q)))
    assert np.isfinite(out[0][1]).all()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("precision,mrt,iso", [("fp64", True, False), ("fp32dev", False, False),
                                               ("fp32sr", True, False), ("mixed", False, False),
                                               ("fp32dev", True, True), ("fp64", False, True)])
def test_batch_strips_equal_tiles(precision, mrt, iso):
    """A batch of 640^2 sites or more marches in strips unless tiles are asked
    for; grids narrower than a strip, of one strip and of many, through a graph
    of steps and single steps, against the two sweeps bit for bit."""
    require_gpu()
    from paper_1907_13415_amd import lc
    shapes = [(400, 500), (333, 301), (64, 70), (600, 56), (57, 9), (300, 350)]
    print("batch strips %s mrt %d iso %d" % (precision, mrt, iso), flush=True)
    params = [(1.0, 2.6 + 0.03 * k, 0.05, 0.3, 0.7, 1.0 + 0.1 * k) for k in range(len(shapes))]
    q5 = [inputs.random_q5((1,) + s, np.random.default_rng(k), amp=0.05) for k, s in enumerate(shapes)]
    out = []
    for tiles in (None, (4, 0), "tuned"):
        b = lc.BatchSolver(precision, shapes, params)
        if tiles == (4, 0):
            b.set_tiles(*tiles)
        if mrt:
            b.set_collision(lc.LC_COLL_MRT, RATES)
        if iso:
            b.set_stencil(lc.LC_STENCIL_ISOTROPIC)
        for k, q in enumerate(q5):
            b.load(k, q)
        if tiles == "tuned":
            b.autotune(1)
            for k, q in enumerate(q5):
                b.load(k, q)
        b.step(67)
        out.append([(b.export(k, lc.LC_FIELD_F), b.export(k, lc.LC_FIELD_Q)) for k in range(len(shapes))])
    for k in range(len(shapes)):
        assert np.isfinite(out[0][k][1]).all()
        for other in out[1:]:
            assert np.array_equal(out[0][k][0], other[k][0]) and np.array_equal(out[0][k][1], other[k][1]), shapes[k]
