"""The Krylov step's first norm, ||f - K u||, comes from its first product: at the
smallest degrees (0: no fused pass follows; 1 and 2), with loads and displacements
on fixed DOFs too (identity rows, whose residual is part of the norm), on voxel
and plane grids.  Oracle: the monomial least-squares step in FP64; tolerances of
the Krylov parity tests."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle.grid import Grid as OGrid
from oracle.operator import assemble_K, simp_scale
from oracle.plane import Grid2D, q4_stiffness
from gpu_util import DEV, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deg", [0, 1, 2])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_krylov_first_norm(dim, deg, dtype):
    from paper_2204_06204_amd.grid import Grid, PlaneGrid
    say(f"krylov norm dim={dim} deg={deg} {dtype}")
    og = Grid2D(33, 9) if dim == 2 else OGrid(17, 9, 5)
    rng = np.random.default_rng(5)
    mask = (rng.random(og.ndof) < 0.1).astype(np.uint8)
    g = PlaneGrid(33, 9, fixed_mask=mask) if dim == 2 else Grid(17, 9, 5, fixed_mask=mask, rho_min=1e-3)
    rho_t = dev(synth.uniform_density(og.E, 3, 0.3, 1.0), dtype)
    s = simp_scale(host(rho_t), 3.0, 0.0 if dim == 2 else 1e-3)
    K = assemble_K(og, s, mask, KE=q4_stiffness()) if dim == 2 else assemble_K(og, s, mask)
    f = host(dev(rng.standard_normal(og.ndof), dtype))
    u0 = host(dev(rng.standard_normal(og.ndof), dtype))
    u = dev(u0, dtype)
    info = torch.zeros(8, dtype=torch.float64, device=DEV)
    g.inner_solve(rho_t, dev(f, dtype), u, deg, method="krylov", omega=1.0, info=info)
    ref, _ = oracle.krylov_step_ref(lambda v: K @ v, f, u0, deg)
    tol = 1e-9 if dtype == torch.float64 else 3e-4
    assert np.abs(host(u) - ref).max() <= tol * np.abs(ref - u0).max()
