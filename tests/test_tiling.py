"""The tilings of the step kernels on the host, and the two-step kernel on
the highest bands of rows."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_two_step_tiles_cover_every_row_once(tmp_path):
    exe = tmp_path / "tiling_check"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2408_15654_amd", "csrc"),
                           os.path.join(ROOT, "tests", "tiling_check.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and "tiling ok" in out.stdout, (out.returncode, out.stdout)


@pytest.mark.gpu
def test_two_steps_on_a_band_of_many_rows():
    """8 x 2 400 000 float32: rows times chunks of a band pass 2^31.  A tile
    height set by the caller selects one step per launch, with the same
    arithmetic of a site, hence no tolerance."""
    from paper_2408_15654_amd import lbm, workloads as W

    nx, ny = 8, 2400000
    rng = np.random.default_rng(8)
    p = W.base_params(nx, ny, walls_y=1, u_wall_top=0.02, r=2.0, rhoA=3.0, muA=0.3, beta=0.3,
                      M=0.05, D=0.02, precision="fp32")
    wave = np.sin(0.37 * np.arange(ny))[:, None]
    fields = (0.5 + 0.4 * wave + 1e-3 * rng.standard_normal((ny, nx)),
              0.2 + 0.1 * wave + 1e-3 * rng.standard_normal((ny, nx)),
              1e-3 * rng.standard_normal((ny, nx)), 1e-3 * rng.standard_normal((ny, nx)))
    got = []
    for rows in (0, 16):
        sim = lbm.Simulation(p)
        sim.set_tile_rows(rows)
        sim.init_fields(*fields)
        sim.step(4)
        got.append(sim.read_fields())
        sim.close()
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k
