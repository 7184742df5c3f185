"""The default z-chunks of the 3D sweeps, which follow from the number of
tiles: every chunk gives the same state bit for bit, so the default must equal
one chunk over the whole depth, at depths below, at and beyond the planes a
block marches, and with a second block on every CU (the last shape), whose
ring points other waves take."""
import numpy as np
import pytest

from paper_1907_13415_amd import inputs
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

PARAMS = (1.0, 2.72, 0.05, 0.3, 0.7, 1.3)


@pytest.mark.parametrize("precision,stencil,variant", [("fp32dev", 0, 2), ("fp64", 0, 2), ("mixed", 0, 2),
                                                       ("fp32dev", 1, 2), ("fp64", 1, 2), ("fp32dev", 0, 3)])
@pytest.mark.parametrize("shape", [(1, 9, 33), (2, 8, 64), (17, 24, 20), (130, 9, 40), (60, 64, 64)])
def test_default_chunk_equals_whole_depth(precision, stencil, variant, shape):
    require_gpu()
    from paper_1907_13415_amd import lc
    print("chunks %s %s stencil %d variant %d" % (shape, precision, stencil, variant), flush=True)
    q5 = inputs.random_q5(shape, np.random.default_rng(11), amp=0.1)
    out = []
    for planes in (0, shape[0]):
        s = lc.Solver("D3Q19", precision, shape, PARAMS)
        s.set_variant(variant)
        s.set_stencil(stencil)
        s.set_chunk(planes)
        s.load(q5)
        s.step(3)
        out.append((s.export(lc.LC_FIELD_F), s.export(lc.LC_FIELD_Q)))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
