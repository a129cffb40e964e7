"""Pairs of steps run where they should, counted; and the kernels that only
large lists and grids reach, bit for bit against single steps.

A batch or pool whose populations exceed 192 MiB sweeps with streaming stores
and keeps the strips of a workgroup in step, also where they belong to
instances of uneven sizes or to slots that have ended."""
import numpy as np
import pytest

from test_gpu_sweep import FIXED, IMPROVED, LLKC, MC, make, same

pytestmark = pytest.mark.gpu


def boxes(nx, ny, period, radius):
    """A closed box with square obstacles."""
    m = np.zeros((ny, nx), np.uint8)
    yy, xx = np.mgrid[0:ny, 0:nx]
    if period:
        m[(abs(xx % period - period // 2) <= radius) & (abs(yy % period - period // 2) <= radius)] = 1
    m[0, :] = m[-1, :] = 1
    m[:, 0] = m[:, -1] = 1
    return m


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("bc", [MC, LLKC, IMPROVED, FIXED])
@pytest.mark.parametrize("nx,ny,kind", [(1009, 521, "open"), (899, 601, "both"), (1121, 547, "x"), (671, 783, "y"), (1233, 601, "closed"),
                                        (64, 32, "both"), (203, 97, "closed"), (392, 364, "open")])
def test_grids_that_run_in_pairs(nx, ny, kind, bc, storage):
    from paper_2009_12584_amd import Simulation

    mask, a, b, per = make(nx, ny, kind)
    prm = dict(bc=bc, G=2.5, Gw=-0.3, periodic=per, storage=storage)
    with Simulation(mask, a, b, **prm) as s:
        s.step(9)
        assert s.pair_steps == 8
    with Simulation(mask, a, b, graph_steps=4, diag_every=8, **prm) as s:  # a graph of two pairs, one of single steps
        s.step(16)
        assert s.launch_counts()["graph_steps"] == 16 and s.pair_steps == 8
    with Simulation(mask, a, b, lanes=2, **prm) as s:
        s.step(9)
        assert s.pair_steps == 0


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("nx,ny,period,radius", [(1024, 700, 32, 7), (700, 500, 20, 6), (64, 8001, 0, 0)])
def test_grids_full_of_walls_run_single_steps(nx, ny, period, radius, storage):
    """In the improved scheme, and the same as the two-lane step."""
    from paper_2009_12584_amd import Simulation

    mask = boxes(nx, ny, period, radius)
    a = 0.5 + 0.2 * np.random.default_rng(2).random((ny, nx))
    x = Simulation(mask, a, 1.0 - a, bc=IMPROVED, storage=storage)
    y = Simulation(mask, a, 1.0 - a, bc=IMPROVED, storage=storage, lanes=2)
    for n in (4, 3):
        x.step(n)
        y.step(n)
        same(x, y)
    assert x.pair_steps == 0
    x.close()
    y.close()


@pytest.mark.parametrize("bc", [MC, LLKC])
@pytest.mark.parametrize("storage,nx,ny,kind", [("f32", 1400, 1001, "closed"), ("f32", 2011, 1403, "both"), ("f32", 2011, 1403, "closed"),
                                                ("f16", 2401, 1681, "both"), ("f16", 2633, 1931, "both"), ("f16", 2633, 1931, "closed")])
def test_single_component_pairs(storage, nx, ny, kind, bc):
    """In the caches and beyond them, against calls of one step each."""
    from paper_2009_12584_amd import Simulation

    mask, a, _, per = make(nx, ny, kind)
    prm = dict(tau=0.9, G=-5.0, bc=bc, Gw=-3.0, periodic=per, storage=storage, model=1, rho0=1.0)
    x = Simulation(mask, 0.2 + 1.5 * a, None, **prm)
    y = Simulation(mask, 0.2 + 1.5 * a, None, **prm)
    for n in (2, 5):
        x.step(n)
        for _ in range(n):
            y.step(1)
        same(x, y)
    assert x.pair_steps == 6 and y.pair_steps == 0
    x.close()
    y.close()


def items(scale):
    """Instances of every rule and border kind, a narrow and a small one among them."""
    out = []
    for k, (nx, ny, kind, bc) in enumerate([(1001, 403, "closed", IMPROVED), (64, 513, "x", MC), (903, 411, "both", IMPROVED),
                                            (1020, 401, "open", LLKC), (333, 503, "y", FIXED), (130, 32, "closed", IMPROVED),
                                            (701, 301, "closed", MC)]):
        if nx > 200:
            nx, ny = int(nx * scale), int(ny * scale)
        mask, a, b, per = make(nx, ny, kind, seed=k)
        out.append((mask, a, b, dict(tau=0.9 + 0.1 * k, G=2.5, bc=bc, Gw=-0.3, chiA=0.4, chiB=0.6, avg=k % 2, periodic=per)))
    return out


def streams(its, storage):
    bytes_per_node = 144 if storage == "f32" else 80
    return sum(m.shape[0] * (-(-m.shape[1] // 64) * 64) * bytes_per_node for m, _, _, _ in its) > 192 << 20


@pytest.mark.parametrize("graph", [0, 12])
@pytest.mark.parametrize("storage,scale,streaming", [("f32", 1.0, True), ("f16", 1.0, False), ("f16", 1.4, True)])
def test_batches_in_pairs(storage, scale, streaming, graph):
    from paper_2009_12584_amd import Batch

    its = items(scale)
    assert streams(its, storage) == streaming
    x = Batch(its, storage=storage, graph_steps=graph)
    y = Batch(its, storage=storage, lanes=2)
    for n in (13, 14):
        x.step(n)
        y.step(n)
        for k in range(x.n):
            for p, q in zip(x.fields(k), y.fields(k)):
                assert np.isfinite(p).all()
                np.testing.assert_array_equal(p, q)
            np.testing.assert_array_equal(x.get_state(k), y.get_state(k))
    assert x.pair_steps == 24 and y.pair_steps == 0
    x.close()
    y.close()


@pytest.mark.parametrize("storage,scale", [("f32", 1.0), ("f16", 1.4)])
def test_pools_in_pairs(storage, scale):
    """Slots of uneven step counts; the first advances with a small request only, the others join later."""
    from paper_2009_12584_amd import Pool, Simulation

    its, steps = items(scale), [33, 9, 18, 31, 1, 46, 23]
    pool = Pool(2 << 30, 8, storage=storage)
    slots = {5: pool.admit(*its[5][:3], steps[5], **its[5][3])}
    pool.advance(8)
    assert pool.pair_steps == 0  # too little fluid
    for k in (0, 1, 2, 3, 4, 6):
        slots[k] = pool.admit(*its[k][:3], steps[k], **its[k][3])
    for _ in range(4):
        pool.advance(11)
    assert 20 <= pool.pair_steps <= 36
    for k, (m, a, b, p) in enumerate(its):
        ref = Simulation(m, a, b, storage=storage, lanes=2, **p)
        ref.step(steps[k])
        for f, g in zip(pool.fields(slots[k]), ref.fields()):
            np.testing.assert_array_equal(f, g)
        ref.close()
    pool.close()
