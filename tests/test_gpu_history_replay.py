"""A captured step holds its place in the Adams-Bashforth sequence (it was captured on a grid with a
history), but not the grid's history: replayed after fields were written without one it takes zeros,
whatever an earlier run, here one of NaN, has left.  The reference is the same grid given a history of
zeros and stepped eagerly: bitwise equal."""
import numpy as np
import pytest

from paper_1803_09563_amd import inputs

from harness import gpu_grid, gpu_state, to_dev
from test_gpu_parity import _wl

pytestmark = pytest.mark.gpu

FIELDS = ("u", "v", "w", "p", "B", "hist")


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1803_09563_amd  # noqa: F401  (fails loudly without libevp.so)
    yield


def _grids(shape, walls, models, mixed, seed, stream):
    """Per model: a grid on `stream`, the reference grid, its fields and a history of zeros and of NaN."""
    import paper_1803_09563_amd as evp
    out = []
    for m, model in enumerate(models):
        wl = _wl(*shape, walls, model)
        f = to_dev(*inputs.random_state(wl.shape, seed + m, walls=walls))
        zero, bad = to_dev(np.zeros((9,) + wl.shape), np.full((9,) + wl.shape, np.nan))
        G, R = (gpu_grid(wl, precision=evp.MIXED if mixed else evp.FP64, stream=s) for s in (stream, None))
        out.append((G, R, f, zero, bad))
    return out


def _capture(run, stream):
    import torch
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        run()
    return g


def _replay(g):
    import torch
    torch.cuda.synchronize()      # the replay runs on the current stream, the grids on their own
    g.replay()
    torch.cuda.synchronize()


def _equal(G, R, fields=FIELDS):
    a, b = gpu_state(R, fields), gpu_state(G, fields)
    for k in fields:
        assert np.isfinite(a[k]).all() and np.array_equal(a[k], b[k]), k


# one block a tile and many; both precisions; several models in one launch (mixed) and one launch each
@pytest.mark.parametrize("shape,walls,models,mixed", [((20, 12, 10), False, ("saramito",), False), ((24, 13, 10), True, ("fene_p",), False),
                                                      ((192, 96, 96), False, ("oldroyd_b",), False), ((20, 12, 10), False, ("saramito",), True),
                                                      ((30, 13, 10), True, ("saramito", "fene_p", "oldroyd_b"), True),
                                                      ((16, 16, 16), False, ("saramito", "fene_p", "oldroyd_b"), False)])
def test_replayed_steps_after_a_write_without_history(shape, walls, models, mixed):
    import torch
    import paper_1803_09563_amd as evp
    s = torch.cuda.Stream()
    cases = _grids(shape, walls, models, mixed, 40, s)
    gs, rs = [c[0] for c in cases], [c[1] for c in cases]
    for G, _, f, _, bad in cases:
        G.write_fields(*f, bad)
    g = _capture(lambda: evp.step_batch(gs, 1e-3, 2), s)
    for _ in range(2):
        for G, _, f, _, bad in cases:
            G.write_fields(*f, bad)
        _replay(g)
        for G, R, f, zero, _ in cases:
            G.write_fields(*f)
            R.write_fields(*f, zero)
        for _ in range(3):        # the second and third replays go on with the history of the first
            _replay(g)
            evp.step_batch(rs, 1e-3, 2)
            for G, R, *_ in cases:
                _equal(G, R)


# Without polymer viscosity the velocities do not depend on B, so that a graph of a single step, which
# always reads the same one of the two buffers of B, can be replayed step after step.
@pytest.mark.parametrize("mixed", [False, True])
def test_replays_of_a_single_step_keep_the_history(mixed):
    import torch
    s = torch.cuda.Stream()
    ((G, R, f, zero, bad),) = _grids((20, 12, 10), False, ("oldroyd_b",), mixed, 41, s)
    for X in (G, R):
        X.set_rheology(0, 1.0, 0.01, 0.0, 1.0)
    G.write_fields(*f, bad)
    g = _capture(lambda: G.step(1e-3, 1), s)
    G.step(1e-3, 1)               # the parity of the capture again
    G.write_fields(*f)
    R.write_fields(*f, zero)
    for _ in range(4):
        _replay(g)
        R.step(1e-3, 1)
        _equal(G, R, ("u", "v", "w", "p"))


# A capture alone makes the host count a history, though nothing has run: eager steps then take zeros too.
def test_eager_steps_after_a_capture_without_replay():
    import torch
    s = torch.cuda.Stream()
    ((G, R, f, zero, bad),) = _grids((20, 12, 10), False, ("saramito",), False, 42, s)
    G.write_fields(*f, bad)
    G.write_fields(*f)
    R.write_fields(*f, zero)
    _capture(lambda: G.step(1e-3, 2), s)
    for _ in range(2):
        G.step(1e-3, 1)
        R.step(1e-3, 1)
        _equal(G, R)
