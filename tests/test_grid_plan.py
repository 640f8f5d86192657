"""Which grids the plane sweep takes, and that its plans cover them within the
kernels' limits (host code, no GPU)."""
import random

import pytest

from . import grid_plan

THIN = [(4, 4, 187500), (5, 5, 300000), (8, 8, 46875), (8, 8, 100000)]
NEAR = [(131, 97, 67), (64, 64, 88), (3, 300, 900), (640, 641, 2), (20, 20, 2500), (256, 256, 256)]


@pytest.mark.parametrize("g", THIN + [(10, 10, 30000), (12, 12, 6944)])
def test_thin_packed_grids_stay_with_the_rows(g):
    assert not grid_plan.takes(7, g, packed=True)


@pytest.mark.parametrize("g", THIN + [(1, 1, 4000000), (2, 2, 200000), (32, 1, 250000), (400000, 1, 1), (110, 1, 9090)])
def test_thin_matrix_free_grids_stay_with_the_bricks(g):
    assert not grid_plan.takes(7, g)


@pytest.mark.parametrize("g", [(1, 1, 4000000), (32, 1, 31250)])
def test_thin_27(g):
    assert not grid_plan.takes(27, g)


@pytest.mark.parametrize("g", [(1, 1, 4000000), (8, 8, 46875), (300, 3, 1111), (100, 2, 5000), (1732, 1733, 1)])
def test_thin_variable_coefficients_stay_with_the_bricks(g):
    assert not grid_plan.takes(1, g)


@pytest.mark.parametrize("g", NEAR)
@pytest.mark.parametrize("npts", [7, 27])
def test_the_others_do_not(npts, g):
    assert grid_plan.takes(npts, g) and grid_plan.takes(npts, g, packed=True)


@pytest.mark.parametrize("npts,g", [(7, (71, 71, 71)), (1, (91, 92, 93)), (1, (256, 256, 256)),
                                    (7, (1 << 14, 1 << 14, 1)), (7, (0, 5, 5))])
def test_sizes_outside_the_range(npts, g):
    assert not grid_plan.takes(npts, g)


def test_half_empty_tiles_of_four_points_take_two():
    assert grid_plan.shape(7, (16, 16, 31250)).points == 2
    assert grid_plan.shape(7, (256, 256, 256)).points == 4


@pytest.mark.parametrize("g", [(272, 272, 272), (400, 400, 400), (250, 250, 250), (800, 800, 100), (912, 913, 24),
                               (72, 72, 1800), (10000, 900, 1), (2300000, 4, 1)])
@pytest.mark.parametrize("npts", [7, 27])
def test_large_grids_are_cut_into_whole_lines(npts, g):
    assert grid_plan.shape(npts, g).W % 16 == 0


@pytest.mark.parametrize("g,takes", [((272, 272, 272), True), ((401, 401, 401), False), ((350, 350, 350), False),
                                     ((720, 360, 100), False), ((256, 256, 256), True), ((201, 201, 201), True)])
def test_matrix_free_cg_of_large_grids(g, takes):
    assert grid_plan.takes_cg(7, g) == takes and grid_plan.takes_cg(27, g)


def test_plans():
    """Tiles and chunks cover the grid; the tile, its ring and the LDS planes fit."""
    rng = random.Random(3)
    for _ in range(4000):
        n = int(10 ** rng.uniform(5.6, 8.3))
        nx = max(1, int(n ** rng.uniform(0, 1)))
        ny = max(1, int((n / nx) ** rng.uniform(0, 1)))
        g = (nx, ny, max(1, n // (nx * ny)))
        for npts in (1, 7, 27):
            if not grid_plan.takes(npts, g):
                continue
            s = grid_plan.shape(npts, g)
            assert (s.ntx - 1) * s.W < nx <= s.ntx * s.W and (s.nty - 1) * s.H < ny <= s.nty * s.H, g
            assert (s.ncz - 1) * s.zb < g[2] <= s.ncz * s.zb, g
            assert s.points in (2, 4) and s.W * s.H <= 256 * s.points and 2 * (s.W + 2) + 2 * s.H <= 256, g
            assert 0 < s.fill <= 1
            assert grid_plan.takes(npts, g, packed=True) == (s.fill >= 0.375) or npts == 1, g
