"""Batches of several kernel variants, which run side by side in chunks of
four steps or more: each simulation gives bit for bit what it gives alone, for
chunks on both sides of that line, over more captured graphs than are kept,
with members leaving and joining, and with two batches on streams of their
own.  The kernels and their order within a simulation are the same, hence no
tolerance."""
import numpy as np
import pytest
import torch

from paper_2408_15654_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu

PRECISIONS = ("fp32", "fp64", "fp16dev")


def problem(i):
    pr = W.random_small(700 + i, nx=40 + 23 * (i % 5), ny=16 + 7 * (i % 4), walls=bool(i & 1),
                        r=(1.0, 0.0, 2.0)[i // 3 % 3], precision=PRECISIONS[i % 3], steps=1)
    return dict(pr.params, precision=PRECISIONS[i % 3]), pr.fields0


def assert_alone(batch, sid, i, steps):
    p, f = problem(i)
    sim = lbm.Simulation(p)
    sim.init_fields(*f)
    sim.step(steps)
    want, got = sim.read_fields(), batch.read_fields(sid)
    for k in want:
        assert np.array_equal(got[k], want[k]), (i, k, steps)
    sim.close()


@pytest.mark.parametrize("chunk", [3, 4, 5])
@pytest.mark.parametrize("count", [2, 3, 9])
def test_side_by_side_equals_alone(chunk, count):
    b = lbm.Batch(1 << 26, max_instances=16)
    b.set_schedule(chunk=chunk)
    ids = [b.submit(problem(i)[0], *problem(i)[1], 20 + i) for i in range(count)]
    b.step(11)
    assert_alone(b, ids[1], 1, 11)
    b.retire(ids[1])  # the places in the tile list change
    ids[1] = b.submit(problem(1)[0], *problem(1)[1], 21)
    b.step(40)
    for i, sid in enumerate(ids):
        assert_alone(b, sid, i, 20 + i)
    b.close()


def test_more_graphs_than_are_kept():
    b = lbm.Batch(1 << 26, max_instances=16)
    b.set_schedule(chunk=64)
    ids = [b.submit(problem(i)[0], *problem(i)[1], 1000) for i in range(9)]
    done = 0
    for k in range(1, 25):
        b.step(k)
        done += k
    for i, sid in enumerate(ids):
        assert_alone(b, sid, i, done)
    b.close()


def test_two_batches_on_their_own_streams():
    batches = []
    for k in range(2):
        with torch.cuda.stream(torch.cuda.Stream()):
            b = lbm.Batch(1 << 26, max_instances=16)
            batches.append((b, [b.submit(problem(i)[0], *problem(i)[1], 100) for i in range(6)]))
    for n in (6, 9, 2, 12):
        for b, _ in batches:
            b.step(n)
    for b, ids in batches:
        for i, sid in enumerate(ids):
            assert_alone(b, sid, i, 29)
        b.close()
