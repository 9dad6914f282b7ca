"""The Krylov step of plane grids at the edges of its 32 x 8 node tiles: one
tile and less, one node more along each axis, and more tiles than blocks (the
blocks then loop over tiles); random fixed DOFs on the tile borders too.
Oracle: the monomial least-squares step in FP64; tolerances of the plane Krylov
parity test."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle.operator import assemble_K, simp_scale
from oracle.plane import Grid2D, q4_stiffness
from gpu_util import DEV, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1, 1), (30, 6), (31, 7), (32, 8), (33, 15), (700, 501)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_plane_krylov_tiles(nx, ny, dtype):
    from paper_2204_06204_amd.grid import PlaneGrid
    say(f"plane krylov {nx}x{ny} {dtype}")
    og = Grid2D(nx, ny)
    rng = np.random.default_rng(nx + ny)
    mask = (rng.random(og.ndof) < 0.05).astype(np.uint8)
    for j in range(ny + 1):
        mask[2 * og.node(0, j):2 * og.node(0, j) + 2] = 1
    g = PlaneGrid(nx, ny, fixed_mask=mask)
    rho_t = dev(synth.uniform_density(og.E, 3, 0.3, 1.0), dtype)
    K = assemble_K(og, simp_scale(host(rho_t), 3.0, 0.0), mask, KE=q4_stiffness())
    f = host(dev(np.where(mask == 0, rng.standard_normal(og.ndof), 0.0), dtype))
    u0 = host(dev(np.where(mask == 0, rng.standard_normal(og.ndof), 0.0), dtype))
    for deg in (1, 2, 4) if og.ndof > 8 else (1,):
        u = dev(u0, dtype)
        info = torch.zeros(8, dtype=torch.float64, device=DEV)
        g.inner_solve(rho_t, dev(f, dtype), u, deg, method="krylov", omega=1.0, info=info)
        ref, _ = oracle.krylov_step_ref(lambda v: K @ v, f, u0, deg)
        tol = 1e-9 if dtype == torch.float64 else 3e-4
        assert np.abs(host(u) - ref).max() <= tol * np.abs(ref - u0).max(), deg
        rn = np.linalg.norm(f - K @ host(u))
        assert abs(host(info)[0] - rn) <= (1e-8 if dtype == torch.float64 else 1e-3) * rn
