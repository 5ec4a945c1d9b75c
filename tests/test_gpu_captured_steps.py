"""lbm_step under HIP graph capture: replays of captured steps, with reads of
the fields between them, give the fields of as many steps taken eagerly.  The
kernels are the same, hence no tolerance."""
import numpy as np
import pytest
import torch

from paper_2408_15654_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu


def problem(nx, ny, precision, flow):
    if flow == "prescribed":
        pr = W.e2_convection(nx=nx, R=nx / 5.0, r=1.0, precision=precision)
        return pr.params, pr.fields0
    pr = W.random_small(41, nx=nx, ny=ny, walls=False, r=1.0, precision=precision, steps=1)
    return dict(pr.params, precision=precision), pr.fields0


# several steps per launch (small grids: up to three, large ones: two) and one;
# captures that together take an even number of steps, so that they can be
# replayed in turn
@pytest.mark.parametrize("captures", [(2,), (4,), (8,), (3, 1), (7, 5)])
@pytest.mark.parametrize("nx,ny,precision,flow", [
    (64, 64, "fp16dev", "ns"), (64, 64, "fp32", "ns"), (40, 40, "fp64", "prescribed"),
    (130, 101, "fp64", "ns"), (400, 390, "fp64", "ns"), (672, 640, "fp32", "ns")])
def test_replayed_steps_equal_eager_steps(nx, ny, precision, flow, captures):
    p, fields = problem(nx, ny, precision, flow)
    stream = torch.cuda.Stream()
    replayed, eager = lbm.Simulation(p, stream=stream), lbm.Simulation(p)
    for sim in (replayed, eager):
        sim.init_fields(*fields)
    graphs = []
    for n in captures:
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1], stream=stream):
            replayed.step(n)
    for _ in range(4):
        for g, n in zip(graphs, captures):
            with torch.cuda.stream(stream):
                g.replay()
            eager.step(n)
        replayed.moments()
        a, b = replayed.read_fields(), eager.read_fields()
        for k in a:
            assert np.array_equal(a[k], b[k]), k
    replayed.close()
    eager.close()
