"""CPU checks of the rules that choose a grid's kernel and launch shape
(lc_launch.h, compiled for the host): every form gives the same values bit for
bit, so the GPU tests that compare forms rest on these to know which ones ran."""
import ctypes
import os
import subprocess

import pytest

import test_gpu_fused2d
from paper_1907_13415_amd import lc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILES, PAIRS, STRIPS = range(3)


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rules") / "rules.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(ROOT, "tests", "native", "launch_rules.cpp"),
                    "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.rule_tiles2d.restype = ctypes.c_int64
    return lib


def grid2d(nx, ny, precision="fp32dev"):
    return lc.make_grid(lc.LC_D2Q9, lc.PRECISIONS[precision], nx, ny, 1)


def ref(g):
    return ctypes.byref(g)


def test_forms_of_the_compared_grids(rules):
    """The grids that the GPU test compares cover pairs, every shape of tile
    with one tile per CU, more tiles than CUs, and strips."""
    seen = set()
    for nx, ny in test_gpu_fused2d.SHAPES:
        g = grid2d(nx, ny)
        form, shape = rules.rule_form2d(ref(g), 0, 0), rules.rule_shape2d(ref(g))
        fits = rules.rule_tiles2d(ref(g), 4) <= rules.rule_num_cu()
        seen.add((form, shape if form == TILES and fits else None))
    assert seen == {(PAIRS, None), (TILES, 1), (TILES, 2), (TILES, 3), (TILES, 4), (TILES, None), (STRIPS, None)}


@pytest.mark.parametrize("nx,ny,form", [(256, 128, PAIRS), (257, 128, TILES), (640, 640, STRIPS), (640, 639, TILES),
                                        (64, 6400, TILES), (74, 12000, TILES), (112, 4000, STRIPS), (616, 664, TILES),
                                        (616, 665, STRIPS)])
def test_form_at_its_thresholds(rules, nx, ny, form):
    """256 and 257 tiles of 16x8; 640^2 sites; strips filled to less than three
    quarters (64 of 112 columns) and more (74 of 112 not, 112 of 112)."""
    assert rules.rule_form2d(ref(grid2d(nx, ny)), 0, 0) == form


def test_steps_that_are_not_paired(rules):
    g, d = grid2d(64, 64), grid2d(64, 64, "fp64")
    assert [rules.rule_form2d(ref(g), i, t) for i, t in ((0, 0), (1, 0), (0, 1))] == [PAIRS, PAIRS, TILES]
    assert [rules.rule_form2d(ref(d), i, t) for i, t in ((0, 0), (1, 0), (0, 1))] == [PAIRS, TILES, TILES]


@pytest.mark.parametrize("precision,nx,ny,variant", [
    ("fp64", 400, 380, lc.LC_VARIANT_FUSED), ("fp64", 448, 448, lc.LC_VARIANT_SPLIT),
    ("fp32dev", 448, 448, lc.LC_VARIANT_FUSED),
    ("fp32sr", 639, 640, lc.LC_VARIANT_FUSED), ("fp64", 640, 640, lc.LC_VARIANT_FUSED),
    ("fp64", 639, 640, lc.LC_VARIANT_SPLIT), ("fp32dev", 64, 7000, lc.LC_VARIANT_SPLIT),
    # more tiles than CUs: full and nearly empty rounds, tiles of one row, narrow grids
    ("fp32dev", 512, 512, lc.LC_VARIANT_FUSED), ("fp64", 512, 512, lc.LC_VARIANT_FUSED),
    ("mixed", 400, 400, lc.LC_VARIANT_FUSED), ("fp64", 742, 256, lc.LC_VARIANT_SPLIT),
    ("fp32sr", 120000, 1, lc.LC_VARIANT_SPLIT), ("fp32dev", 300000, 1, lc.LC_VARIANT_SPLIT),
    ("fp64", 11111, 9, lc.LC_VARIANT_FUSED), ("mixed", 10000, 2, lc.LC_VARIANT_FUSED),
    ("fp64", 33, 4454, lc.LC_VARIANT_FUSED), ("mixed", 16, 9187, lc.LC_VARIANT_FUSED),
    ("fp32dev", 8, 37500, lc.LC_VARIANT_FUSED), ("fp64", 29400, 5, lc.LC_VARIANT_SPLIT)])
def test_auto_variant_at_its_thresholds(rules, precision, nx, ny, variant):
    assert rules.rule_auto_variant(ref(grid2d(nx, ny, precision)), 0) == variant


def test_batch_of_the_strip_test_marches(rules):
    """The batch that the GPU test compares with two sweeps is one that
    marches by default, and the small one of the other batch tests is not."""
    big = [(400, 500), (333, 301), (64, 70), (600, 56), (57, 9), (300, 350)]
    small = [(23, 37), (64, 64), (40, 96), (16, 16), (70, 130)]
    for shapes, takes in ((big, 1), (small, 0)):
        arr = (lc.lc_grid * len(shapes))(*[grid2d(nx, ny) for ny, nx in shapes])
        assert rules.rule_march_takes(len(shapes), arr) == takes


@pytest.mark.parametrize("threads,tx,ty", [(1024, 32, 20), (1024, 16, 8), (768, 16, 16), (768, 40, 4)])
@pytest.mark.parametrize("nx,ny", [(1, 1), (301, 419), (1, 65535), (61000, 65535), ((1 << 27) - 32, 5), (1 << 27, 5),
                                   ((1 << 27) + 1, 29), (1 << 28, 4), (89478485, 1), (89478500, 40), (1 << 30, 3)])
def test_tiles_of_any_grid_fit_their_launches(rules, threads, tx, ty, nx, ny):
    """Fewer than 2^32 threads along x in every launch; the launches take the
    tile columns one after another, each once; rows that fit take one."""
    out = (ctypes.c_int64 * 256)()
    n = rules.rule_tile_launches(ref(grid2d(nx, ny)), tx, ty, threads, out)
    ntx, nty = -(-nx // tx), -(-ny // ty)
    column = 0
    for k in range(n):
        bx, by, xb, before = out[4 * k:4 * k + 4]
        assert bx * threads < 1 << 32 and by == nty and xb == column * tx and before == column * nty
        column += bx
    assert column == ntx and (n == 1 or ntx * threads >= 1 << 32)


# one tile per CU and more: the smallest tile with the fewest rounds
SHAPE_OF = {(9000, 7): 1, (20000, 7): 1, (12000, 5): 1, (400, 400): 2, (70, 2000): 2, (448, 448): 3, (33, 4000): 3,
            (540, 540): 4, (100, 100): 0, (256, 256): 1, (301, 419): 4}


@pytest.mark.parametrize("nx,ny", SHAPE_OF)
def test_tile_shape_has_the_fewest_rounds(rules, nx, ny):
    g = grid2d(nx, ny)
    rounds = [-(-rules.rule_tiles2d(ref(g), v) // rules.rule_num_cu()) for v in range(5)]
    shape = rules.rule_shape2d(ref(g))
    assert shape == rounds.index(min(rounds)) == SHAPE_OF[nx, ny]


SWEEPS, SINGLE = lc.LC_VARIANT_SPLIT, lc.LC_VARIANT_FUSED


@pytest.mark.parametrize("precision,iso,nx,ny,variant", [
    # strips that nearly fill, or just overfill, the waves the chip holds
    ("fp64", 0, 65000, 7, SWEEPS), ("mixed", 0, 65000, 7, SWEEPS), ("fp64", 0, 60000, 8, SWEEPS),
    ("fp64", 1, 65000, 7, SWEEPS), ("fp64", 0, 1075 * 56, 64, SWEEPS), ("mixed", 0, 522 * 56, 64, SWEEPS),
    ("fp32dev", 1, 1044 * 56, 16, SWEEPS), ("fp32sr", 0, 1126 * 56, 8, SWEEPS),
    # full rounds, many rounds, FP32, tiles with idle rows
    ("fp64", 0, 1003 * 56, 8, SINGLE), ("fp64", 0, 2027 * 56, 16, SINGLE), ("fp64", 0, 65000, 9, SINGLE),
    ("fp64", 0, 410000, 1, SINGLE), ("mixed", 0, 410000, 1, SINGLE), ("fp32dev", 0, 65000, 7, SINGLE),
    ("fp32dev", 0, 1044 * 56, 16, SINGLE), ("fp64", 0, 501 * 56, 64, SINGLE), ("fp64", 0, 640, 640, SINGLE),
    ("mixed", 0, 1000, 1000, SINGLE), ("fp64", 1, 700, 700, SINGLE), ("fp64", 0, 56, 8000, SINGLE),
    ("fp64", 0, 2048, 2048, SINGLE), ("fp32sr", 0, 640, 640, SINGLE)])
def test_strips_only_where_they_beat_the_sweeps(rules, precision, iso, nx, ny, variant):
    """As measured: on grids of very many columns a march over the whole
    height leaves the chip part empty in its last round."""
    g = grid2d(nx, ny, precision)
    assert rules.rule_march_takes(1, ref(g)) == 1
    assert rules.rule_auto_variant(ref(g), iso) == variant


def test_batch_of_wide_short_grids_takes_the_sweeps(rules):
    """60 grids of 2048x7: 2220 strips for 1024 waves."""
    arr = (lc.lc_grid * 60)(*[grid2d(2048, 7, "mixed")] * 60)
    assert rules.rule_march_takes(60, arr) == 1 and rules.rule_march_beats_sweeps(60, arr, 0) == 0
    arr = (lc.lc_grid * 64)(*[grid2d(300, 300, "mixed")] * 64)
    assert rules.rule_march_beats_sweeps(64, arr, 0) == 1


@pytest.mark.parametrize("nx,ny,shape", [(4096, 3, 0), (4097, 3, 1), (30000, 3, 1), (5120, 8, 1), (5200, 8, 0), (30000, 9, 0),
                                         (256, 256, 0), (1, 4000, 0), (2048, 2048, 0)])
def test_reverse_tiles_of_few_rows(rules, nx, ny, shape):
    """40x4 tiles where they go through the chip in fewer rounds than 16x16."""
    assert rules.rule_rev_shape(ref(grid2d(nx, ny, "fp64"))) == shape


def test_regions_that_wrap_once(rules):
    """The rule that spares a tile's halo region the division, against the
    coordinates themselves: never where one is beyond the next period, and on
    every grid at least as wide as the tile."""
    for t in (4, 8, 16, 32, 64, 128):
        for n in list(range(1, 3 * t + 3)) + [1 << 20, 1 << 30]:
            x0s = range(0, n, t) if n < 1 << 20 else (0, (n - 1) // t * t)
            once = all(-n <= x0 - 2 and x0 + t + 1 < 2 * n for x0 in x0s)
            rule = rules.rule_region_wraps_once(n, t) == 1
            assert rule == once, (n, t)
            assert once or n < t


@pytest.mark.parametrize("nz,tiles,margin,chunk", [(2000, 15, 0.08, 63), (2000, 15, 0.0, 59), (33, 380, 0.08, 17),
                                                   (500, 32, 0.08, 63), (96, 36, 0.08, 14), (256, 256, 0.08, 64),
                                                   (1, 1, 0.08, 1), (64, 1, 0.08, 1)])
def test_chunks_of_the_3d_single_pass(rules, nz, tiles, margin, chunk):
    """Shorter chunks in more blocks only where the estimate is clearly in
    their favour, even ones of the longest otherwise."""
    assert rules.rule_pick_chunk(nz, tiles, 64, 8, 1, ctypes.c_double(margin)) == chunk


@pytest.mark.parametrize("nz,planes,chunk", [(200, 33, 29), (200, 128, 100), (200, 100, 100), (200, 1, 1), (200, 200, 200),
                                             (33, 8, 7), (7, 2**31 - 1, 7), (65535, 65534, 32768), (1, 5, 1)])
def test_chunks_asked_for_are_cut_evenly(rules, nz, planes, chunk):
    """As many chunks as asked for, none longer, none much shorter."""
    assert rules.rule_even_chunk(nz, planes) == chunk
    assert -(-nz // chunk) == -(-nz // min(planes, nz)) and chunk <= planes


def test_batch_launch_needs_a_batch():
    for call, args in ((lc.lc_batch_get_launch, ()), (lc.lc_batch_set_strips, (1,))):
        with pytest.raises(lc.LCError) as e:
            call(None, *args)
        assert e.value.code == lc.LC_EINVAL
