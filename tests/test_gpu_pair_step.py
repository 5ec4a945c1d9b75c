"""Two time steps per launch on large grids: the row-walking two-step kernel
gives bit for bit what one step per launch gives (a tile height set by the
caller selects the latter).  The arithmetic of a site is the same in both,
hence no tolerance."""
import numpy as np
import pytest

from paper_2408_15654_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu


# strips of 56 columns, bands of ny / 8 rows: whole and one column over, even
# and odd, rows that do not divide, bands of two rows (tiles of one), a band's
# chunks more than its rows, tiles of several rounds
@pytest.mark.parametrize("precision,nx,ny,walls", [
    ("fp32", 672, 640, False), ("fp32", 673, 641, True), ("fp32", 727, 650, True),
    ("fp32", 30001, 17, False), ("fp32", 30000, 17, True), ("fp32", 64, 8200, True),
    ("fp32", 3001, 3000, False), ("fp64", 560, 512, False), ("fp64", 561, 515, True),
    ("fp64", 20001, 16, True), ("fp64", 1023, 769, False)])
@pytest.mark.parametrize("r,ratio", [(1.0, 10.0), (2.0, 1.0)])
def test_two_steps_equal_single_steps(precision, nx, ny, walls, r, ratio):
    rng = np.random.default_rng(nx + ny)
    p = W.base_params(nx, ny, walls_y=int(walls), u_wall_bot=-0.01 * walls,
                      u_wall_top=0.02 * walls, r=r, rhoA=ratio, muA=0.1 * ratio, beta=0.3,
                      gx=1e-6, gy=-2e-6, M=0.05, D=0.02, precision=precision)
    # a drop across the periodic corner (or on the bottom wall), noise elsewhere
    phi, th = W.single_drop(nx, ny, min(nx, ny) / 3.0, cx=2.0, cy=3.0, periodic_y=not walls)
    phi = phi + 1e-3 * rng.standard_normal(phi.shape)
    psi = 0.4 * (1.0 + 0.4 * np.cos(th)) * W.unit_peak(phi)
    u = 1e-3 * rng.standard_normal((2, ny, nx))
    two, one = lbm.Simulation(p), lbm.Simulation(p)
    one.set_tile_rows(2)
    for sim in (two, one):
        sim.init_fields(phi, psi, u[0], u[1])
    for n in (4, 7):
        for sim in (two, one):
            sim.step(n)
        a, b = two.read_fields(), one.read_fields()
        for k in a:
            assert np.array_equal(a[k], b[k]), (n, k, float(np.abs(a[k] - b[k]).max()))
        one.set_state(two.get_state())  # the previous velocity among it
    for sim in (two, one):
        sim.close()
