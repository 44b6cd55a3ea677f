"""Edges of the FP64 predictor's tiles (16 x 8 and 32 x 8 cells, chunks of z planes, 16-byte pairs
staged into LDS): grids narrower than a tile and its halo, widths and heights that leave a remainder,
every wall row a tile can start or end at, chunks of one plane, and batches whose chunks differ from a
single grid's.  Stage parity with the oracle 1e-12, as for the predictor elsewhere."""
import numpy as np
import pytest

import oracle
from paper_1803_09563_amd import inputs

from harness import assert_close, gpu_grid, gpu_state, oracle_solver, oracle_state, to_dev
from test_gpu_parity import _wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1803_09563_amd  # noqa: F401  (fails loudly without libevp.so)
    yield


def _stage(shape, model, walls, seed=91):
    nx, ny, nz = shape
    wl = _wl(nx, ny, nz, walls, model, force=(inputs.FORCE_SIN_X_OF_Y, 0.7, 2.0),
             wall_velocity=(0.2, -0.1, 0.05, 0.3) if walls else (0.0, 0.0, 0.0, 0.0))
    u, v, w, B = inputs.random_state(wl.shape, seed, walls=walls)
    hist = 0.1 * np.random.default_rng(seed + 1).standard_normal((9,) + wl.shape)
    return wl, (u, v, w, B, hist)


# 8 and 10: the halo wraps more than once round a 16-wide tile; 20, 40, 48: remainders; 96 x 96 x 48
# and 128 x 64 x 32: the 32-wide tile
@pytest.mark.parametrize("model", ["saramito", "fene_p"])
@pytest.mark.parametrize("shape", [(8, 8, 8), (10, 20, 10), (40, 12, 8), (48, 10, 12), (96, 96, 48), (128, 60, 32)])
def test_periodic_tiles(shape, model):
    wl, fields = _stage(shape, model, False)
    s = oracle_solver(wl)
    s.write_fields(*fields)
    s.step(1e-3, 1, flags=oracle.Solver.STOP_AFTER_PREDICTOR)
    G = gpu_grid(wl)
    G.write_fields(*to_dev(*fields))
    G.step(1e-3, 1, flags=2)
    assert_close(oracle_state(s), gpu_state(G, ("u", "v", "w", "B")), 1e-12, f"{shape} {model}")


# ny from one partial tile to a last tile of one, two, ... rows: the ghost rows beyond the top wall
# come from rows of the tile or from its halo
@pytest.mark.parametrize("model", ["saramito", "fene_p"])
@pytest.mark.parametrize("ny", [4, 5, 7, 8, 9, 10, 11, 13, 16, 17, 18, 19])
def test_wall_rows_of_a_tile(ny, model):
    wl, fields = _stage((24, ny, 10), model, True)
    s = oracle_solver(wl)
    s.write_fields(*fields)
    s.step(1e-3, 1, flags=oracle.Solver.STOP_AFTER_PREDICTOR)
    G = gpu_grid(wl)
    G.write_fields(*to_dev(*fields))
    G.step(1e-3, 1, flags=2)
    assert_close(oracle_state(s), gpu_state(G, ("u", "v", "w", "B")), 1e-12, f"ny={ny} {model}")


@pytest.mark.parametrize("walls", [False, True])
def test_batch_chunks_equal_single_bitwise(walls):
    import paper_1803_09563_amd as evp
    singles, batched = [], []
    for b in range(24):
        wl, fields = _stage((48, 24, 48), ("saramito", "fene_p", "oldroyd_b")[b % 3], walls, seed=100 + b)
        a, c = gpu_grid(wl), gpu_grid(wl)
        for G in (a, c):
            G.write_fields(*to_dev(*fields))
        a.step(1e-3, 3)
        singles.append(a)
        batched.append(c)
    evp.step_batch(batched, 1e-3, 3)
    for a, c in zip(singles, batched):
        sa, sc = gpu_state(a), gpu_state(c)
        for k in sa:
            assert np.array_equal(sa[k], sc[k]), k


# The mixed form (FP32 stresses): widths that are and are not multiples of 4 (groups of 16 bytes or single
# values), narrow and wide tiles, every wall-row remainder class.  Stored values are rounded to 6e-8 and
# dt times right-hand sides of up to 10^2, themselves good to 1e-6, adds 1e-7: 5e-6 leaves a factor of 20.
@pytest.mark.parametrize("model", ["saramito", "fene_p"])
@pytest.mark.parametrize("shape,walls", [((8, 8, 8), False), ((10, 20, 10), False), ((30, 12, 8), False), ((40, 12, 8), False),
                                         ((96, 96, 48), False), ((128, 64, 40), False), ((10, 9, 8), True), ((24, 8, 10), True),
                                         ((24, 13, 10), True), ((48, 17, 10), True), ((128, 75, 64), True)])
def test_mixed_tiles(shape, walls, model):
    import paper_1803_09563_amd as evp
    wl, fields = _stage(shape, model, walls)
    s = oracle_solver(wl)
    s.write_fields(*fields)
    s.step(1e-3, 1, flags=oracle.Solver.STOP_AFTER_PREDICTOR)
    G = gpu_grid(wl, precision=evp.MIXED)
    G.write_fields(*to_dev(*fields))
    G.step(1e-3, 1, flags=2)
    assert_close(oracle_state(s), gpu_state(G, ("u", "v", "w", "B")), 5e-6, f"{shape} {model} mixed")


# a grid's numbers do not depend on its tile and chunk: alone a 48^3 grid runs in narrow tiles, a batch
# of 24 of them in wide ones
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("adv", [0, 1])
def test_mixed_batch_tiles_equal_single_bitwise(adv, walls):
    import paper_1803_09563_amd as evp
    singles, batched = [], []
    for b in range(24):
        wl, fields = _stage((48, 48, 48), ("saramito", "fene_p", "oldroyd_b", "oldroyd_b")[b % 4], walls, seed=200 + b)
        wl.adv, wl.kappa = adv, 1e-3 * (b & 1)
        if b % 4 == 3:
            wl.model = evp.NEO_HOOKEAN
        a, c = gpu_grid(wl, precision=evp.MIXED), gpu_grid(wl, precision=evp.MIXED)
        for G in (a, c):
            G.write_fields(*to_dev(*fields))
        a.step(1e-3, 2)
        singles.append(a)
        batched.append(c)
    evp.step_batch(batched, 1e-3, 2)
    for a, c in zip(singles, batched):
        sa, sc = gpu_state(a), gpu_state(c)
        for k in sa:
            assert np.array_equal(sa[k], sc[k]), k


# the kernel for several models in its narrow tiles, with rows in groups of 16 bytes and value by value
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("shape", [(16, 12, 10), (10, 12, 8)])
def test_models_in_one_launch_equal_single_bitwise(shape, walls):
    import paper_1803_09563_amd as evp
    singles, batched = [], []
    for b in range(4):
        wl, fields = _stage(shape, ("saramito", "fene_p", "oldroyd_b", "oldroyd_b")[b], walls, seed=300 + b)
        if b == 3:
            wl.model = evp.NEO_HOOKEAN
        a, c = gpu_grid(wl, precision=evp.MIXED), gpu_grid(wl, precision=evp.MIXED)
        for G in (a, c):
            G.write_fields(*to_dev(*fields))
        a.step(1e-3, 2)
        singles.append(a)
        batched.append(c)
    evp.step_batch(batched, 1e-3, 2)
    for a, c in zip(singles, batched):
        sa, sc = gpu_state(a), gpu_state(c)
        for k in sa:
            assert np.array_equal(sa[k], sc[k]), k
