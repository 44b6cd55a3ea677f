"""Edges of the projection's kernels against the oracle's plain definition."""
import numpy as np
import pytest

import oracle
from paper_1803_09563_amd import inputs

from harness import assert_close, gpu_grid, gpu_state, oracle_solver, to_dev
from test_gpu_parity import _wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1803_09563_amd  # noqa: F401  (fails loudly without libevp.so)
    yield


# Wall heights where the segmented tridiagonal solve changes its block shape or has a last segment of
# one row or of all rows but one.  The tolerance grows as the condition number of the lowest modes,
# (ny / 256)^2, from 1e-12 at 256 rows.
@pytest.mark.parametrize("ny", [15, 16, 255, 257, 271, 512, 513, 1009])
def test_segments_of_the_wall_solve(ny):
    nx, nz = 16, 10
    wl = _wl(nx, ny, nz, True, "oldroyd_b")
    u, v, w, B = inputs.random_state(wl.shape, 5, walls=True)
    s = oracle_solver(wl)
    s.write_fields(u, v, w, B)
    ru, rv, rw, rp = oracle.project(s.g, s.u, s.v, s.w, 1.0, s.r.rho)
    G = gpu_grid(wl)
    G.write_fields(*to_dev(u, v, w, B))
    G.project()
    assert_close({"u": ru, "v": rv, "w": rw, "p": rp}, gpu_state(G, ("u", "v", "w", "p")),
                 1e-12 * max(1.0, (ny / 256) ** 2), f"ny={ny}")


# Line transforms of one, two, three and four radices in each direction, and lengths so short that a
# block takes several tiles and its last one fewer.  Tolerance as above.
@pytest.mark.parametrize("shape", [(8, 10, 12), (10, 8, 8), (12, 30, 10), (20, 12, 24), (48, 8, 30), (160, 10, 8),
                                   (10, 240, 12), (8, 12, 320), (12, 8, 512), (30, 384, 8), (480, 8, 10)])
def test_line_lengths_of_the_transforms(shape):
    nx, ny, nz = shape
    wl = _wl(nx, ny, nz, False, "oldroyd_b")
    u, v, w, B = inputs.random_state(wl.shape, 6, walls=False)
    s = oracle_solver(wl)
    s.write_fields(u, v, w, B)
    ru, rv, rw, rp = oracle.project(s.g, s.u, s.v, s.w, 1.0, s.r.rho)
    G = gpu_grid(wl)
    G.write_fields(*to_dev(u, v, w, B))
    G.project()
    assert_close({"u": ru, "v": rv, "w": rw, "p": rp}, gpu_state(G, ("u", "v", "w", "p")),
                 1e-12 * max(1.0, (max(shape) / 256) ** 2), f"{shape}")


# Single grids of few square planes, which take the fused plane transforms.  Tolerance as above.
@pytest.mark.parametrize("n", [8, 10, 12, 16, 20, 24, 30, 32, 40, 48, 60, 64])
@pytest.mark.parametrize("nz", [8, 30])
def test_plane_transforms_of_few_planes(n, nz):
    wl = _wl(n, n, nz, False, "oldroyd_b")
    u, v, w, B = inputs.random_state(wl.shape, 7, walls=False)
    s = oracle_solver(wl)
    s.write_fields(u, v, w, B)
    ru, rv, rw, rp = oracle.project(s.g, s.u, s.v, s.w, 1.0, s.r.rho)
    G = gpu_grid(wl)
    G.write_fields(*to_dev(u, v, w, B))
    G.project()
    assert_close({"u": ru, "v": rv, "w": rw, "p": rp}, gpu_state(G, ("u", "v", "w", "p")), 1e-12, f"{n}x{n}x{nz}")
