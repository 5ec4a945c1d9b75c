"""Several time steps per launch (grids too small to fill the device): the
block kernel gives bit for bit what one step per launch gives.

A tile height set by the caller selects one launch of the single-step kernel
per step, so the two paths are compared on the same inputs.  The arithmetic
of a site is the same in both, hence no tolerance."""
import numpy as np
import pytest

from paper_2408_15654_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu


def assert_equal(params, fields, steps, label):
    block, single = lbm.Simulation(params), lbm.Simulation(params)
    single.set_tile_rows(1)
    for sim in (block, single):
        sim.init_fields(*fields)
    for n in steps:  # separate calls: odd and even numbers of launches
        for sim in (block, single):
            sim.step(n)
        a, b = block.read_fields(), single.read_fields()
        for k in a:
            assert np.array_equal(a[k], b[k]), (label, n, k, float(np.abs(a[k] - b[k]).max()))
        # the whole state, the previous velocity among it: saved after the
        # block launches and continued by single steps
        single.set_state(block.get_state())
    for sim in (block, single):
        sim.close()


# sizes around the sites a block keeps with 1, 2 and 3 steps (12..14, 8..10,
# 4..6), one column or row short and over, smaller than a block, odd and even;
# the larger ones take 2 steps, 1 step, and two rounds of blocks
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev"])
@pytest.mark.parametrize("nx,ny,walls", [(3, 3, False), (4, 3, True), (6, 10, True), (7, 5, False),
                                         (16, 16, False), (19, 31, True), (60, 61, False),
                                         (61, 60, True), (130, 101, True), (150, 141, False),
                                         (206, 190, True), (301, 260, False)])
def test_block_steps_equal_single_steps(precision, nx, ny, walls):
    rng = np.random.default_rng(nx * 1000 + ny)
    for r, ratio, eos in ((1.0, 1.0, "linear"), (2.0, 3.0, "langmuir"), (1.0, 10.0, "linear")):
        p = W.base_params(nx, ny, walls_y=int(walls), u_wall_bot=-0.01 * walls,
                          u_wall_top=0.02 * walls, r=r, rhoA=ratio, muA=0.1 * ratio, beta=0.3,
                          eos=eos, gx=1e-6, gy=-2e-6, M=0.05, D=0.02, precision=precision)
        phi, th = W.single_drop(nx, ny, min(nx, ny) / 3.0, periodic_y=not walls)
        psi = 0.4 * (1.0 + 0.4 * np.cos(th)) * W.unit_peak(phi)
        u = 1e-3 * rng.standard_normal((2, ny, nx))
        assert_equal(p, (phi, psi, u[0], u[1]), (1, 2, 3, 4, 7),
                     f"{precision} {nx}x{ny} r={r} ratio={ratio}")


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev"])
@pytest.mark.parametrize("nx,r", [(40, 1.0), (101, 2.0), (150, 0.0)])
def test_block_steps_with_a_prescribed_velocity(precision, nx, r):
    pr = W.e2_convection(nx=nx, R=nx / 5.0, r=r, precision=precision)
    assert_equal(pr.params, pr.fields0, (1, 2, 5, 6), f"{precision} {nx} r={r}")


def test_nonfinite_in_a_block_is_reported():
    """A value that overflows inside a launch of several steps raises the
    flag, as in a single step."""
    pr = W.c1_stationary_drop()
    p = dict(pr.params, precision="fp16dev", fp16_scale=(2.0 ** 30, 0.0, 0.0))
    sim = lbm.Simulation(p)
    sim.init_fields(*pr.fields0)
    sim.step(3)
    with pytest.raises(lbm.NonFiniteError):
        sim.moments()
    sim.close()
