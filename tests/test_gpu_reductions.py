"""The domain sums of lbm_moments and lbm_shape at the sizes where the number
of reduction blocks changes (256 sites a block, at most 1024 blocks), against
sums of the fields that lbm_read_fields returns."""
import math

import numpy as np
import pytest

from paper_2408_15654_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (17, 15), (16, 16), (257, 1 + 256), (512, 512),
                                   (513, 512), (1024, 513)])
def test_sums_of_the_fields(precision, nx, ny):
    phi, th = W.single_drop(nx, ny, min(nx, ny) / 4.0)
    p = W.base_params(nx, ny, rhoA=3.0, muA=0.3, beta=0.2, precision=precision)
    rng = np.random.default_rng(nx + ny)
    u = 1e-3 * rng.standard_normal((2, ny, nx))
    sim = lbm.Simulation(p)
    sim.init_fields(phi, (1 + 0.5 * np.cos(th)) * W.unit_peak(phi), u[0], u[1])
    sim.step(2)
    m, sh, f = sim.moments(), sim.shape(), sim.read_fields()
    sim.close()
    # rho of Eq. (15) and the products are formed with a few roundings each;
    # a sum of n values in any order is within n 2^-53 of the sum of their
    # magnitudes (n + 8 covers both)
    rho = p["rhoB"] + (p["rhoA"] - p["rhoB"]) * f["phi"]
    u2 = f["ux"] ** 2 + f["uy"] ** 2
    want = {"sum_phi": f["phi"], "sum_psi": f["psi"], "mom_x": rho * f["ux"],
            "mom_y": rho * f["uy"], "kinetic": 0.5 * rho * u2}
    for k, v in want.items():
        bound = (nx * ny + 8) * 2.0 ** -53 * math.fsum(np.abs(v).ravel())
        assert abs(m[k] - math.fsum(v.ravel())) <= bound, k
    assert abs(m["max_u"] - math.sqrt(u2.max())) <= 4 * 2.0 ** -53 * m["max_u"]
    assert m["step"] == 2 and m["nonfinite"] == 0
    bound = (nx * ny + 8) * 2.0 ** -53 * math.fsum(np.abs(f["phi"]).ravel())
    assert abs(sh["area"] - math.fsum(f["phi"].ravel())) <= bound


def test_shape_reports_a_lost_state():
    pr = W.c1_stationary_drop()
    sim = lbm.Simulation(dict(pr.params, precision="fp16dev", fp16_scale=(2.0 ** 30, 0, 0)))
    sim.init_fields(*pr.fields0)
    sim.step(2)
    with pytest.raises(lbm.NonFiniteError):
        sim.shape()
    with pytest.raises(lbm.LbmError) as e:
        sim.step(1)
    assert e.value.status == lbm.LBM_ESTATE
    sim.close()
