"""Launches captured by the caller between plain steps, against a simulation of single steps, bit for bit.

A captured launch reads the buffer that held the state when it was captured.
Any even number of plain steps, and a state set at a time of the same parity,
leave the state in that buffer, whether the steps run in pairs or not."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GRIDS = [(1233, 601), (203, 97)]  # strip sweeps; pair tiles


def simulations(nx, ny, storage, stream):
    from paper_2009_12584_amd import Simulation

    rng = np.random.default_rng(7)
    yy, xx = np.mgrid[0:ny, 0:nx]
    mask = np.zeros((ny, nx), np.uint8)
    mask[yy <= 0.2 * (xx - nx / 2) + ny / 8] = 1
    mask[0, :] = mask[-1, :] = 1
    mask[:, 0] = mask[:, -1] = 1
    a = np.where((xx - nx * 0.4) ** 2 + (yy - ny * 0.5) ** 2 <= (ny * 0.3) ** 2, 1.0, 0.055) * (1.0 + 0.05 * rng.random((ny, nx)))
    b = (1.11 - np.minimum(a, 1.05)) * (1.0 + 0.05 * rng.random((ny, nx)))
    prm = dict(bc=2, G=2.5, chiA=0.4, chiB=0.6, storage=storage, stream=stream)
    return Simulation(mask, a, b, **prm), Simulation(mask, a, b, lanes=2, **prm)


def captured(stream, body):
    import torch

    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        body()
    torch.cuda.synchronize()

    def replay():
        with torch.cuda.stream(stream):  # in order with the handle's own work
            g.replay()

    return replay


def same(x, y):
    for p, q in zip(x.fields(), y.fields()):
        assert np.isfinite(p).all()
        np.testing.assert_array_equal(p, q)


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("nx,ny", GRIDS)
@pytest.mark.parametrize("before", [0, 1, 2])
def test_plain_steps_between_replays(nx, ny, storage, before):
    import torch

    st = torch.cuda.Stream()
    x, y = simulations(nx, ny, storage, st)
    x.step(before)
    y.step(before)
    six = captured(st, lambda: x.step(6))
    for k, n in enumerate((2, 6, 1, 3, 10, 5, 2)):
        if k == 3:
            four = captured(st, lambda: x.step(4))  # a second graph, captured later
        six()
        y.step(6)
        same(x, y)
        if k >= 3:
            four()
            y.step(4)
            same(x, y)
        x.step(n)
        y.step(n)
        same(x, y)
        if n % 2:  # back to the parity that the graphs were captured at
            x.step(1)
            y.step(1)
    x.close()
    y.close()


@pytest.mark.parametrize("nx,ny", GRIDS)
@pytest.mark.parametrize("before", [1, 2])
def test_states_set_between_replays(nx, ny, before):
    import torch

    st = torch.cuda.Stream()
    x, y = simulations(nx, ny, "f32", st)
    x.step(before)
    y.step(before)
    six = captured(st, lambda: x.step(6))
    six()
    y.step(6)
    for step in (8, 40):  # times of the parity at the capture, when before is even; of the other, when it is odd
        buf, _ = y.get_state()
        x.set_state(buf, step)
        if (step - before) % 2:
            x.step(1)
            y.step(1)
        six()
        y.step(6)
        same(x, y)
        x.step(2)
        y.step(2)
        six()
        y.step(6)
        same(x, y)
    x.close()
    y.close()


@pytest.mark.parametrize("nx,ny", GRIDS)
def test_captured_fields_follow_plain_steps(nx, ny):
    import torch

    st = torch.cuda.Stream()
    x, y = simulations(nx, ny, "f32", st)
    x.step(2)
    y.step(2)
    out = [torch.zeros(ny, nx, device="cuda") for _ in range(4)]
    look = captured(st, lambda: x.fields_device(*out))
    for n in (2, 4, 6, 10):
        x.step(n)
        y.step(n)
        look()
        torch.cuda.synchronize()
        for p, q in zip(out, y.fields()):
            np.testing.assert_array_equal(p.cpu().numpy().astype(np.float64), q)
    x.close()
    y.close()
