"""Every variant of the kernels that take several steps per launch (r != 1 or
not, rho_A != rho_B or not, both equations of state, each storage) against
one step per launch, which a tile height set by the caller selects; and that
it is those kernels that run.  The arithmetic of a site is the same in both,
hence no tolerance."""
import numpy as np
import pytest

from paper_2408_15654_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu

VARIANTS = [(r, ratio) for r in (1.0, 2.0) for ratio in (1.0, 10.0)]


def params(nx, ny, walls, r, ratio, eos, precision, **kw):
    return W.base_params(nx, ny, walls_y=int(walls), u_wall_bot=-0.01 * walls,
                         u_wall_top=0.02 * walls, r=r, rhoA=ratio, muA=0.1 * ratio, beta=0.3,
                         eos=eos, gx=1e-6, gy=-2e-6, M=0.05, D=0.02, precision=precision, **kw)


def fields(nx, ny, walls):
    rng = np.random.default_rng(nx + 7 * ny)
    phi, th = W.single_drop(nx, ny, min(nx, ny) / 3.0, cx=2.0, cy=3.0, periodic_y=not walls)
    phi = phi + 1e-3 * rng.standard_normal(phi.shape)
    psi = 0.4 * (1.0 + 0.4 * np.cos(th)) * W.unit_peak(phi)
    u = 1e-3 * rng.standard_normal((2, ny, nx))
    return phi, psi, u[0], u[1]


def assert_equal_to_single_steps(p, f, kernel, calls):
    several, single = lbm.Simulation(p), lbm.Simulation(p)
    single.set_tile_rows(2)
    name, steps = several.step_plan()
    assert name.startswith(kernel + "<") and (steps > 1 or kernel == "lbm_step_kernel"), (name, steps)
    assert single.step_plan() == (single.step_kernel_name(), 1)
    for sim in (several, single):
        sim.init_fields(*f)
    for n in calls:
        for sim in (several, single):
            sim.step(n)
        a, b = several.read_fields(), single.read_fields()
        for k in a:
            assert np.array_equal(a[k], b[k]), (name, n, k, float(np.abs(a[k] - b[k]).max()))
        single.set_state(several.get_state())  # the previous velocity among it
    for sim in (several, single):
        sim.close()
    return name


@pytest.mark.parametrize("eos", ["linear", "langmuir"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev"])
@pytest.mark.parametrize("r,ratio", VARIANTS)
@pytest.mark.parametrize("nx,ny,walls", [(61, 60, True), (92, 75, False)])
def test_block_kernel(nx, ny, walls, r, ratio, precision, eos):
    name = assert_equal_to_single_steps(params(nx, ny, walls, r, ratio, eos, precision),
                                        fields(nx, ny, walls), "lbm_block_kernel", (2, 3, 8, 7))
    storage = {"fp64": "F64C", "fp32": "F32C", "fp16dev": "F16"}[precision]
    variant = [str(v).lower() for v in (r != 1, ratio != 1, True)]
    assert name == "lbm_block_kernel<%s>" % ", ".join([storage] + variant)


# both cache policies of the stores (grids that stay in the caches, and not)
@pytest.mark.parametrize("eos", ["linear", "langmuir"])
@pytest.mark.parametrize("r,ratio", VARIANTS)
@pytest.mark.parametrize("precision,nx,ny,walls,storage", [
    ("fp32", 785, 761, True, "F32C"), ("fp32", 1601, 1300, False, "F32"),
    ("fp64", 561, 515, True, "F64C"), ("fp64", 1101, 1000, False, "F64")])
def test_pair_kernel(precision, nx, ny, walls, storage, r, ratio, eos):
    name = assert_equal_to_single_steps(params(nx, ny, walls, r, ratio, eos, precision),
                                        fields(nx, ny, walls), "lbm_pair_kernel", (4, 7))
    assert name == "lbm_pair_kernel<%s, %s, %s>" % (storage, str(r != 1).lower(),
                                                    str(ratio != 1).lower())


@pytest.mark.parametrize("precision,n", [("fp32", 700), ("fp64", 560)])
@pytest.mark.parametrize("row", [0, 350, -1])
def test_nonfinite_in_a_two_step_launch_is_reported(precision, n, row):
    """A velocity whose square overflows raises the flag; the state is lost
    until it is set again."""
    p, (phi, psi, ux, uy) = params(n, n, False, 1.0, 10.0, "linear", precision), fields(n, n, False)
    sim = lbm.Simulation(p)
    assert sim.step_plan()[0].startswith("lbm_pair_kernel<")
    lost = ux.copy()
    lost[row, 3] = 1e25 if precision == "fp32" else 1e200
    sim.init_fields(phi, psi, lost, uy)
    sim.step(4)
    with pytest.raises(lbm.NonFiniteError):
        sim.moments()
    with pytest.raises(lbm.LbmError) as e:
        sim.step(4)
    assert e.value.status == lbm.LBM_ESTATE
    sim.init_fields(phi, psi, ux, uy)
    sim.step(4)
    assert sim.moments()["nonfinite"] == 0
    sim.close()


@pytest.mark.parametrize("walls", [False, True])
def test_single_steps_of_the_default_plan(walls):
    """2048x1024 float32, one step per call: the default plan of the step
    kernel (2-row tiles, then 1-row tiles at the end of each band) gives the
    bits of 1-row tiles."""
    nx, ny = 2048, 1024
    p, f = params(nx, ny, walls, 1.0, 10.0, "linear", "fp32"), fields(nx, ny, walls)
    default, ones = lbm.Simulation(p), lbm.Simulation(p)
    ones.set_tile_rows(1)
    rows, tail, height = default.tile_plan()
    assert rows > 1 and tail > 0 and height == 1
    for sim in (default, ones):
        sim.init_fields(*f)
    for _ in range(7):
        default.step(1)  # a call of one step is a launch of the step kernel
    ones.step(7)
    a, b = default.read_fields(), ones.read_fields()
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    default.close()
    ones.close()
