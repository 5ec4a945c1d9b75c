"""The short tiles at the end of each XCD's band, on grids whose tiles all run
at once: they never make a second round of wavefronts, and the fields are bit
for bit those of 1-row tiles (a site's arithmetic does not depend on its tile,
hence no tolerance)."""
import numpy as np
import pytest

from paper_2408_15654_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu


# none fits, some fit, all fit, more than one round without them; bands of
# unequal height; two columns per lane and one
@pytest.mark.parametrize("precision,nx,ny", [
    ("fp64", 330, 330), ("fp64", 371, 373), ("fp64", 290, 290), ("fp64", 451, 455),
    ("fp16dev", 640, 640), ("fp16dev", 704, 709), ("fp16dev", 512, 515), ("fp16dev", 639, 641),
    ("fp16dev", 1024, 511), ("fp32", 620, 620)])
@pytest.mark.parametrize("walls", [False, True])
def test_short_tiles_that_fit(precision, nx, ny, walls):
    pr = W.random_small(31, nx=nx, ny=ny, walls=walls, r=1.0, precision=precision, steps=1)
    p = dict(pr.params, precision=precision)
    default, ones = lbm.Simulation(p), lbm.Simulation(p)
    ones.set_tile_rows(1)
    for sim in (default, ones):
        sim.init_fields(*pr.fields0)
        sim.step(5)
    a, b = default.read_fields(), ones.read_fields()
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    rows, tail, height = default.tile_plan()
    assert height == 1 and 0 <= tail <= ny // 8
    default.close()
    ones.close()
