"""Mixed-form Runge-Kutta batches: alone a 32^3 grid runs in narrow tiles, four of its model in wide ones,
whose kernel keeps some registers in memory; a grid's numbers are the same in both."""
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


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("adv", [0, 1])
def test_mixed_rk3_batch_equals_single_bitwise(adv, walls):
    import paper_1803_09563_amd as evp
    singles, batched = [], []
    for b in range(12):
        wl = _wl(32, 32, 32, walls, ("saramito", "fene_p", "oldroyd_b")[b % 3], force=(inputs.FORCE_SIN_X_OF_Y, 0.7, 2.0))
        wl.adv, wl.kappa = adv, 1e-3 * (b & 1)
        f = to_dev(*inputs.random_state(wl.shape, 400 + b, walls=walls))
        a, c = gpu_grid(wl, precision=evp.MIXED), gpu_grid(wl, precision=evp.MIXED)
        for G in (a, c):
            G.set_integrator("rk3")
            G.write_fields(*f)
        a.step(1e-3, 2)
        singles.append(a)
        batched.append(c)
    evp.step_batch(batched, 1e-3, 2)
    for a, c in zip(singles, batched):
        sa, sc = gpu_state(a), gpu_state(c)
        for k in sa:
            assert np.isfinite(sa[k]).all() and np.array_equal(sa[k], sc[k]), k
