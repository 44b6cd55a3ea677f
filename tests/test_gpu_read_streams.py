"""What Grid.read_fields returns may be used on the caller's current stream at once, also where the grid
works on a stream of its own."""
import numpy as np
import pytest

from paper_1803_09563_amd import inputs

from harness import gpu_grid, to_dev
from test_gpu_parity import _wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1803_09563_amd  # noqa: F401  (fails loudly without libevp.so)
    yield


def test_read_fields_are_there_on_the_current_stream():
    import torch
    wl = _wl(128, 128, 64, False, "saramito")
    f = to_dev(*inputs.random_state(wl.shape, 8, amp_u=0.1))
    G = gpu_grid(wl, stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    G.write_fields(*f)
    G.step(1e-3, 40)              # some milliseconds ahead of the read on the grid's stream
    out = G.read_fields(("u", "B"))
    now = {k: t.clone() for k, t in out.items()}
    torch.cuda.synchronize()
    for k, t in out.items():
        assert np.array_equal(now[k].cpu().numpy(), t.cpu().numpy()), k


def test_memory_of_a_dropped_read_waits_for_its_use():
    import torch
    wl = _wl(128, 128, 64, False, "saramito")
    f = to_dev(*inputs.random_state(wl.shape, 9, amp_u=0.1))
    G = gpu_grid(wl, stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    G.write_fields(*f)
    a, b = (torch.randn(8192, 8192, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    t = G.read_fields(("B",))["B"]
    for _ in range(8):
        a = torch.tanh(a @ b)     # the current stream is busy for some ten milliseconds
    got, ptr = t.sum(), t.data_ptr()
    del t
    later = G.read_fields(("B",))["B"]
    assert later.data_ptr() != ptr
    assert got.item() == later.sum().item()
