"""Fields written without a history: the history reads as zero, is saved as zero and is not used by the
next step, whatever an earlier run left in its place; a captured write clears it on every replay."""
import ctypes

import numpy as np
import pytest

from paper_1803_09563_amd import inputs

from harness import gpu_grid, gpu_state, to_dev
from test_gpu_parity import _wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1803_09563_amd  # noqa: F401  (fails loudly without libevp.so)
    yield


def _fields(wl, seed):
    return inputs.random_state(wl.shape, seed, walls=wl.walls)


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_no_history_after_write(precision, walls):
    import paper_1803_09563_amd as evp
    prec = evp.MIXED if precision == "mixed" else evp.FP64
    wl = _wl(20, 13 if walls else 12, 10, walls, "saramito")
    f = to_dev(*_fields(wl, 3))
    bad = to_dev(np.full((9,) + wl.shape, np.nan))[0]
    fresh, used, loaded = (gpu_grid(wl, precision=prec) for _ in range(3))
    fresh.write_fields(*f)
    used.write_fields(*f, bad)
    used.step(1e-3, 1)
    used.write_fields(*f)
    assert not used.read_fields(("hist",))["hist"].any()
    a, b = fresh.save_state(), used.save_state()
    loaded.write_fields(*f, bad)
    loaded.load_state(b)
    assert not loaded.read_fields(("hist",))["hist"].any()
    for G in (fresh, used, loaded):
        G.step(1e-3, 2)
    ref = gpu_state(fresh, ("u", "v", "w", "p", "B", "hist"))
    assert ref["hist"].any()
    for G in (used, loaded):
        got = gpu_state(G, ("u", "v", "w", "p", "B", "hist"))
        for k in ref:
            assert np.array_equal(ref[k], got[k]), k
    assert a.numel() == b.numel()


def test_captured_write_clears_the_history():
    import torch
    wl = _wl(16, 16, 16, False, "oldroyd_b")
    f = to_dev(*_fields(wl, 4))
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    G = gpu_grid(wl, stream=s)
    G.write_fields(*f)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        G.write_fields(*f)
    for _ in range(3):
        G.step(1e-3, 2)
        torch.cuda.synchronize()
        assert G.read_fields(("hist",))["hist"].any()
        g.replay()
        torch.cuda.synchronize()
        assert not G.read_fields(("hist",))["hist"].any()


def test_captured_read_of_the_history_follows_the_grid():
    import torch
    import paper_1803_09563_amd as evp
    wl = _wl(16, 16, 16, False, "oldroyd_b")
    f = to_dev(*_fields(wl, 4))
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    G = gpu_grid(wl, stream=s)
    G.write_fields(*f)
    out = torch.empty((9,) + wl.shape, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        assert evp.lib.evp_read_fields(G.handle, evp.READ_HIST, None, None, None, None, None, ctypes.c_void_p(out.data_ptr())) == 0
    for steps in (0, 1, 0, 2):
        if steps:
            G.step(1e-3, steps)
        else:
            G.write_fields(*f)
        torch.cuda.synchronize()      # the replay runs on the current stream, the grid on its own
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, G.read_fields(("hist",))["hist"])
        assert bool(out.any()) == (steps > 0)
