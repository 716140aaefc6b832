"""The map kernel's split of a block's galaxies among waves and workgroups, and
its three classes of galaxies (inside every aperture of the block, in some,
in none), against the binary64 oracle: n_in equal everywhere, map and SNR
within the bound of the binary32 filter arithmetic (1e-4 of sum Q |eps| / n_gal,
see test_gpu_aperture)."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_aperture import _check

pc = pytest.importorskip("paper_1208_3658_amd")
pytestmark = pytest.mark.gpu


@pytest.fixture(params=[1, 2], ids=["8x8_blocks", "16x16_blocks"])
def points_per_lane(request):
    pc.pc_debug_ap_points_per_lane(request.param)
    yield request.param
    pc.pc_debug_ap_points_per_lane(0)


# runs of 1 to 64 galaxies (groups of four and remainders), one to thousands of
# runs, one block (sixteen workgroups) to more blocks than are split at all
@pytest.mark.parametrize("n,nx,ny,theta", [
    (1, 1, 1, 5.0), (3, 3, 2, 5.0), (5, 8, 8, 0.6), (64, 9, 8, 5.0), (67, 17, 16, 2.0), (4099, 33, 7, 40.0),
    (30011, 40, 50, 2.0), (3001, 300, 310, 1.0), (900, 1032, 1040, 0.7)])
def test_runs_and_parts(n, nx, ny, theta, points_per_lane):
    cat, side = synth.shear_catalog(n, density=35.0, config=5)
    grid = (0.01 * side, -0.02 * side, side / nx, side / ny, nx, ny)
    ref = oracle.aperture_grid(cat, grid, theta, 35.0)
    _check(pc.pc_aperture_mass(cat, grid, theta, 35.0), ref, 35.0)


@pytest.mark.parametrize("theta", [0.4, 1.7, 6.0])
def test_galaxies_at_the_limits_of_the_classes(theta, points_per_lane):
    """Galaxies at theta, and by up to 1e-4 of it nearer or farther, from
    corners of blocks, and near the blocks' edges."""
    nx, ny, dx, dy = 61, 54, 0.05, 0.07
    grid = (-1.0, 2.0, dx, dy, nx, ny)
    rng = np.random.default_rng(8)
    n, bs = 6000, 8 * points_per_lane
    ix = rng.integers(0, nx // bs, n) * bs + rng.integers(0, 2, n) * (bs - 1)
    iy = rng.integers(0, ny // bs, n) * bs + rng.integers(0, 2, n) * (bs - 1)
    far = rng.choice([0.0, 1e-7, 1e-6, 1e-5, 2e-5, 1e-4], n) * rng.choice([-1.0, 1.0], n)
    r = np.where(rng.random(n) < 0.2, bs * dx * 0.06 * rng.random(n), theta * (1.0 + far))
    ang = rng.choice([0.0, 0.5, 1.0, 1.5, 0.25, 0.81], n) * np.pi
    cat = (-1.0 + ix * dx + r * np.cos(ang), 2.0 + iy * dy + r * np.sin(ang),
           0.2 * rng.standard_normal(n), 0.2 * rng.standard_normal(n))
    ref = oracle.aperture_grid(cat, grid, theta, 35.0)
    _check(pc.pc_aperture_mass(cat, grid, theta, 35.0), ref, 35.0)
