"""Two-step sweeps against single tile steps, bit for bit.

The two-lane step (lanes = 2) never sweeps and is bit-identical to the
one-lane tile step, so it is the reference; the grids are just large enough
for the sweep.  Step counts are odd and even, so runs end on pairs and on
single steps."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

MC, LLKC, IMPROVED, FIXED = range(4)


def make(nx, ny, kind, seed=5):
    """(mask, rhoA0, rhoB0, periodic) of a box that a sweep covers with ragged strips and segments."""
    rng = np.random.default_rng(seed)
    mask = np.zeros((ny, nx), np.uint8)
    yy, xx = np.mgrid[0:ny, 0:nx]
    if kind == "closed":  # inclined plane, solid borders
        mask[yy <= 0.2 * (xx - nx / 2) + ny / 8] = 1
    if kind != "open":  # obstacles next to the borders, a one-node one among them
        mask[(xx - 5) ** 2 + (yy - ny // 2) ** 2 <= 36] = 1
        mask[(xx - nx + 2) ** 2 + (yy - ny // 3) ** 2 <= 100] = 1
        mask[ny - 9, 117 % nx] = 1
    periodic = {"open": 3, "both": 3, "x": 1, "y": 2, "closed": 0}[kind]
    if not periodic & 1:
        mask[:, 0] = mask[:, -1] = 1
    if not periodic & 2:
        mask[0, :] = mask[-1, :] = 1
    a = np.where((xx - nx * 0.4) ** 2 + (yy - ny * 0.5) ** 2 <= (ny * 0.3) ** 2, 1.0, 0.055)
    a = a * (1.0 + 0.05 * rng.random((ny, nx)))
    b = (1.055 - np.minimum(a, 1.0)) * (1.0 + 0.05 * rng.random((ny, nx)))
    return mask, a, b, periodic


def same(x, y):
    fx, fy = x.fields(), y.fields()
    assert all(np.isfinite(f).all() for f in fx)
    for p, q in zip(fx, fy):
        np.testing.assert_array_equal(p, q)
    np.testing.assert_array_equal(x.get_state()[0], y.get_state()[0])


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("bc", [MC, LLKC, FIXED, IMPROVED])
@pytest.mark.parametrize("nx,ny,kind", [(1009, 521, "open"), (899, 601, "both"), (1121, 547, "x"), (671, 783, "y"),
                                        (64, 8001, "both"), (1233, 601, "closed")])
def test_sweeps_equal_single_steps(nx, ny, kind, bc, storage):
    from paper_2009_12584_amd import Simulation

    mask, a, b, per = make(nx, ny, kind)
    prm = dict(tau=0.9, G=2.5, bc=bc, Gw=-0.3, chiA=0.4, chiB=0.6, avg=int(kind == "x"), periodic=per, storage=storage)
    x = Simulation(mask, a, b, **prm)
    y = Simulation(mask, a, b, lanes=2, **prm)
    for n in (2, 1, 7, 4):
        x.step(n)
        y.step(n)
        same(x, y)
    x.close()
    y.close()


@pytest.mark.parametrize("storage,nx,ny", [("f32", 1153, 1231), ("f16", 1801, 1501)])
@pytest.mark.parametrize("bc,kind", [(MC, "both"), (LLKC, "closed"), (IMPROVED, "open")])
def test_streaming_sweeps_equal_single_steps(storage, nx, ny, bc, kind):
    """Beyond the caches the strips of a workgroup keep in step, also where one has fewer rows."""
    from paper_2009_12584_amd import Simulation

    mask, a, b, per = make(nx, ny, kind)
    mask[ny // 2 : ny // 2 + 40, 60:170] = 1  # strips with short segments and with none
    prm = dict(tau=0.9, G=2.5, bc=bc, Gw=-0.3, chiA=0.4, chiB=0.6, periodic=per, storage=storage)
    x = Simulation(mask, a, b, **prm)
    y = Simulation(mask, a, b, lanes=2, **prm)
    for n in (5, 4):
        x.step(n)
        y.step(n)
        same(x, y)
    x.close()
    y.close()


@pytest.mark.parametrize("bc", [MC, IMPROVED])
@pytest.mark.parametrize("graph,diag", [(10, 0), (8, 4), (6, 12), (2, 0), (0, 5)])
def test_sweeps_in_graphs_and_between_diagnostics(graph, diag, bc):
    from paper_2009_12584_amd import Simulation

    mask, a, b, per = make(1233, 601, "closed")
    prm = dict(bc=bc, Gw=-0.2, G=2.5, periodic=per, diag_every=diag)
    x = Simulation(mask, a, b, graph_steps=graph, **prm)
    y = Simulation(mask, a, b, lanes=2, **prm)
    for n in (3, 20, 1, 17):
        x.step(n)
        y.step(n)
        assert x.t == y.t
        same(x, y)
    if graph:
        assert x.launch_counts()["graph_steps"] > 0
    assert x.diag()["mass"] == pytest.approx(y.diag()["mass"], rel=1e-13)
    # resume from a state taken after an odd number of launches
    x.step(2)
    buf, t = x.get_state()
    y.set_state(buf, t)
    x.step(5)
    y.step(5)
    same(x, y)
    x.close()
    y.close()


def test_captured_steps_replay():
    """Steps captured by the caller: an even number returns to the buffer it started from."""
    import torch
    from paper_2009_12584_amd import Simulation

    mask, a, b, per = make(1233, 601, "closed")
    st = torch.cuda.Stream()
    prm = dict(bc=LLKC, Gw=-0.2, G=2.5, periodic=per, stream=st)
    x = Simulation(mask, a, b, **prm)
    y = Simulation(mask, a, b, lanes=2, **prm)
    x.step(2)
    y.step(2)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        x.step(6)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        y.step(6)
        same(x, y)
    x.close()
    y.close()


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("bc", [MC, LLKC, FIXED, IMPROVED])
@pytest.mark.parametrize("nx,ny,kind", [(64, 32, "both"), (64, 47, "y"), (197, 64, "x"), (203, 97, "closed"), (392, 364, "open")])
def test_pair_tiles_equal_single_steps(nx, ny, kind, bc, storage):
    """Small grids: one tile row to the most tiles, ragged tiles, tiles across periodic borders."""
    from paper_2009_12584_amd import Simulation

    mask, a, b, per = make(nx, ny, kind)
    prm = dict(tau=0.9, G=2.5, bc=bc, Gw=-0.3, chiA=0.4, chiB=0.6, avg=int(kind == "x"), periodic=per, storage=storage)
    x = Simulation(mask, a, b, graph_steps=8, **prm)
    y = Simulation(mask, a, b, lanes=2, **prm)
    for n in (2, 1, 17, 6):
        x.step(n)
        y.step(n)
        same(x, y)
    x.close()
    y.close()


@pytest.mark.parametrize("bc", [MC, LLKC])
@pytest.mark.parametrize("storage,nx,ny", [("f32", 1153, 701), ("f16", 1801, 1501)])
@pytest.mark.parametrize("kind", ["both", "closed"])
def test_single_component_sweeps_equal_single_steps(storage, nx, ny, bc, kind):
    """Against calls of one step each, which never sweep."""
    from paper_2009_12584_amd import Simulation

    mask, a, b, per = make(nx, ny, kind)
    prm = dict(tau=0.9, G=-5.0, bc=bc, Gw=-3.0, periodic=per, storage=storage, model=1, rho0=1.0)
    x = Simulation(mask, 0.2 + 1.5 * a, None, **prm)
    y = Simulation(mask, 0.2 + 1.5 * a, None, **prm)
    for n in (2, 5):
        x.step(n)
        for _ in range(n):
            y.step(1)
        same(x, y)
    x.close()
    y.close()


def mixed_items():
    """Instances of every rule and border kind, uneven sizes, together large enough to sweep."""
    out = []
    for k, (nx, ny, kind, bc) in enumerate([(331, 203, "closed", IMPROVED), (64, 257, "x", MC), (455, 187, "both", IMPROVED),
                                            (640, 301, "open", LLKC), (209, 333, "y", FIXED), (130, 32, "closed", IMPROVED)]):
        mask, a, b, per = make(nx, ny, kind, seed=k)
        out.append((mask, a, b, dict(tau=0.9 + 0.1 * k, G=2.5, bc=bc, Gw=-0.3, chiA=0.4, chiB=0.6, avg=k % 2, periodic=per)))
    return out


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("graph,diag", [(0, 0), (10, 0), (0, 9), (12, 6)])
def test_batch_sweeps_equal_single_steps(graph, diag, storage):
    from paper_2009_12584_amd import Batch

    items = [(m, a, b, dict(p, diag_every=diag)) for m, a, b, p in mixed_items()]
    x = Batch(items, storage=storage, graph_steps=graph)
    y = Batch(items, storage=storage, lanes=2)
    for n in (5, 24, 3):
        x.step(n)
        y.step(n)
        for k in range(x.n):
            for p, q in zip(x.fields(k), y.fields(k)):
                assert np.isfinite(p).all()
                np.testing.assert_array_equal(p, q)
            np.testing.assert_array_equal(x.get_state(k), y.get_state(k))
    x.close()
    y.close()


@pytest.mark.parametrize("storage,diag", [("f32", 0), ("f16", 0), ("f32", 7)])
def test_pool_sweeps_stop_each_slot_at_its_step(storage, diag):
    """Slots of uneven step counts, one joining late, against single simulations."""
    from paper_2009_12584_amd import Pool, Simulation

    items, steps = mixed_items(), [31, 6, 18, 31, 1, 23]
    pool = Pool(1 << 30, 8, storage=storage, diag_every=diag)
    slots = [pool.admit(m, a, b, n, **p) for (m, a, b, p), n in zip(items[:5], steps)]
    pool.advance(9)
    slots.append(pool.admit(*items[5][:3], steps[5], **items[5][3]))
    for _ in range(8):
        pool.advance(5)
    for (m, a, b, p), n, slot in zip(items, steps, slots):
        ref = Simulation(m, a, b, storage=storage, lanes=2, **p)
        ref.step(n)
        for f, g in zip(pool.fields(slot), ref.fields()):
            np.testing.assert_array_equal(f, g)
        ref.close()
    pool.close()


@pytest.mark.parametrize("lanes,storage", [(1, "f32"), (1, "f16"), (2, "f32")])
@pytest.mark.parametrize("nx,ny", [(64, 8), (65, 33), (200, 97), (1030, 515)])
def test_reductions_equal_sums_of_the_fields(nx, ny, lanes, storage):
    """One tile, ragged tiles, and more tiles than the last reduction has threads."""
    from paper_2009_12584_amd import Simulation

    mask, a, b, per = make(nx, ny, "x")
    s = Simulation(mask, a, b, tau=0.9, G=2.5, bc=MC, periodic=per, storage=storage, lanes=lanes)
    s.step(3)
    d = s.diag()
    ra, rb, ux, uy = (f.astype(np.float32) for f in s.fields())
    for k, r in enumerate((ra, rb)):  # the reduction's node masses are exact, the fields rounded to 24 bits
        assert d["mass"][k] == pytest.approx(r.sum(dtype=np.float64), rel=2.0**-23)
    for k, u in enumerate((ux, uy)):  # the same terms, added in another order
        t = (ra + rb).astype(np.float64) * u
        assert abs(d["momentum"][k] - t.sum()) <= 2.0**-52 * nx * ny * np.abs(t).sum()
    assert d["max_speed"] == np.sqrt((ux * ux + uy * uy).max().astype(np.float64))
    s.close()
