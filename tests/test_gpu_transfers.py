"""Host transfers (initial fields, fields, checkpoints) at the sizes where
their path changes: one staging chunk (2 MiB in all), several chunks, and
arrays large enough for worker threads (32 MiB); odd sizes, so that chunks end
inside elements' neighbours and scratch planes have gaps."""
import numpy as np
import pytest

from paper_2408_15654_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu

SIZES = [(3, 3), (64, 64), (255, 205), (256, 205), (511, 401), (733, 717), (1025, 1031)]


def problem(nx, ny, precision, **kw):
    rng = np.random.default_rng(nx + ny)
    p = W.base_params(nx, ny, precision=precision, **kw)
    return p, [np.ascontiguousarray(a) for a in (0.5 + 0.4 * rng.random((ny, nx)),
                                                 0.4 * rng.random((ny, nx)),
                                                 *(1e-3 * rng.standard_normal((2, ny, nx))))]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_fields_and_checkpoint_come_back(nx, ny, precision):
    """The initial level reads back as the fields that went in: the psi of
    fluid at the initial equilibrium is the sum of its own populations'
    sources, so the check is on a uniform field per array (each distinct) and
    on a checkpoint that restores random fields bit for bit."""
    p, fields = problem(nx, ny, precision)
    sim = lbm.Simulation(p)
    flat = [np.full((ny, nx), v) for v in (0.75, 0.25, 0.0078125, -0.015625)]
    sim.init_fields(*flat)
    got = sim.read_fields()
    for k, v in zip(("phi", "psi", "ux", "uy"), (0.75, 0.25, 0.0078125, -0.015625)):
        # a uniform state streams into itself; the sums of nine weights are
        # within 16 roundings of it
        eps = 2.0 ** (-53 if precision == "fp64" else -24)
        assert np.abs(got[k] - v).max() <= 16 * eps * max(abs(v), 1.0), k
    sim.init_fields(*fields)
    sim.step(2)
    want, state = sim.read_fields(), sim.get_state()
    other = lbm.Simulation(p)
    other.set_state(state)
    got = other.read_fields()
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    n = int(p["nx"]) * int(p["ny"]) * 26 * (8 if precision == "fp64" else 4)
    assert other.get_state()[:8 + n] == state[:8 + n]
    for sim in (sim, other):
        sim.step(3)
    a, b = sim.read_fields(), other.read_fields()
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    sim.close()
    other.close()


def test_threaded_fields_come_back():
    """Arrays of 34 MB: a prescribed velocity is kept as it is given, so with
    float64 storage it reads back bit for bit."""
    nx, ny = 2111, 2003
    p, fields = problem(nx, ny, "fp64", flow="prescribed")
    sim = lbm.Simulation(p)
    sim.init_fields(*fields)
    got = sim.read_fields()
    assert np.array_equal(got["ux"], fields[2]) and np.array_equal(got["uy"], fields[3])
    sim.close()


@pytest.mark.parametrize("nx,ny", SIZES + [(2111, 2003)])
def test_invalid_initial_values_are_found_anywhere(nx, ny):
    """A NaN, an infinity, or psi >= 1 under the Langmuir law, at the first
    and the last site of an array: refused, and the state before it stays."""
    p, fields = problem(nx, ny, "fp32", eos="langmuir", beta=0.2)
    sim = lbm.Simulation(p)
    sim.init_fields(*fields)
    sim.step(1)
    want = sim.read_fields()
    for field, value in ((0, np.nan), (1, np.inf), (2, -np.inf), (3, np.nan), (1, 1.0)):
        for at in (0, -1):
            bad = [a.copy() for a in fields]
            bad[field].ravel()[at] = value
            with pytest.raises(lbm.LbmError) as e:
                sim.init_fields(*bad)
            assert e.value.status == lbm.LBM_EINVAL
            assert ("psi < 1" in str(e.value)) == (value == 1.0)
    got = sim.read_fields()
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    sim.close()


def test_transfers_from_several_threads():
    """Distinct handles are independent: threads reading and restoring at the
    same time share the staging buffers."""
    import threading

    sims, errors = [], []
    for i in range(4):
        p, fields = problem(500 + 50 * i, 531, "fp32")
        sim = lbm.Simulation(p)
        sim.init_fields(*fields)
        sim.step(2)
        sims.append((sim, sim.read_fields(), sim.get_state()))

    def loop(sim, want, state):
        try:
            for _ in range(5):
                sim.set_state(state)
                got = sim.read_fields()
                assert all(np.array_equal(got[k], want[k]) for k in want)
        except BaseException as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=loop, args=s) for s in sims]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors[0]
    for sim, _, _ in sims:
        sim.close()
