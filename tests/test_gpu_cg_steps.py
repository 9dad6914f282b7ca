"""The CG recurrence at its smallest step counts: one step (no fused pass),
two (one fused pass, the iterate leaves the caller's vector and returns), and
three and four (the iterate alternates between the two workspace vectors, so
the last step reads either of them).  Voxel and plane grids, with one and two
right-hand sides, and the outer step on top (with one load case its last CG
step also forms the sensitivity).  Oracle and tolerances: textbook Jacobi-PCG
in FP64, those of the PCG and outer-step parity tests."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle.grid import Grid as OGrid
from oracle.outer import OuterContext, outer_step_ref
from gpu_util import DEV, dev, host, say

pytestmark = pytest.mark.gpu


def _tol(dtype):
    return 1e-10 if dtype == torch.float64 else 2e-4


@pytest.mark.parametrize("nrhs", [1, 2])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("steps", [1, 2, 3, 4])
def test_pcg_few_steps(steps, dtype, nrhs):
    from paper_2204_06204_amd.grid import Grid
    say(f"pcg steps={steps} {dtype} nrhs={nrhs}")
    p = synth.multiload_cantilever(37, 18, 19, seed=4)
    og = OGrid(p.nx, p.ny, p.nz)
    g = Grid.from_problem(p, max_rhs=nrhs)
    rho = dev(synth.uniform_density(p.E, 3), dtype)
    s = oracle.simp_scale(host(rho), p.penal, p.rho_min)
    K = oracle.assemble_K(og, s, p.fixed_mask)
    D = oracle.jacobi_diag(og, s, p.fixed_mask)
    rng = np.random.default_rng(5)
    u0 = np.where(p.fixed_mask == 0, 0.1 * rng.standard_normal((nrhs, p.ndof)), 0.0)
    u = dev(u0.ravel(), dtype)
    u0 = host(u).reshape(nrhs, -1)
    info = torch.zeros(8 * nrhs, dtype=torch.float64, device=DEV)
    g.inner_solve(rho, dev(p.loads[:nrhs].ravel(), dtype), u, steps, info=info)
    inf = host(info).reshape(nrhs, 8)
    for r, ur in enumerate(host(u).reshape(nrhs, -1)):
        ref, res = oracle.pcg_ref(lambda v: K @ v, D, p.loads[r], u0[r], steps)
        assert np.abs(ur - ref).max() <= _tol(dtype) * np.abs(ref).max()
        assert inf[r][3] == steps and inf[r][4] == 0
        assert abs(inf[r][0] - np.linalg.norm(res)) <= (1e-8 if dtype == torch.float64 else 1e-2) * np.linalg.norm(res)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("steps", [1, 2, 3, 4])
def test_outer_step_few_inner_steps(steps, dtype):
    from paper_2204_06204_amd.grid import Grid
    say(f"outer inner={steps} {dtype}")
    p = synth.cantilever(37, 18, 19, volfrac=0.3, filter_radius=1.5, outer_iters=1, inner_steps=steps, seed=7)
    ctx = OuterContext(p.nx, p.ny, p.nz, p.filter_radius, p.fixed_mask, p.springs)
    F = np.atleast_2d(p.loads[0])
    g = Grid.from_problem(p)
    x = g.project_volume(dev(p.x0, dtype), lo=0.0, hi=1.0, vmax=p.vmax)
    x_ref, u_ref, rec, _ = outer_step_ref(ctx, host(x), np.zeros_like(F), F, 1, 0.002, steps, 0.0, 1.0, p.vmax)
    u = torch.zeros(p.ndof, dtype=dtype, device=DEV)
    info = torch.zeros(8, dtype=torch.float64, device=DEV)
    g.outer_step(x, u, dev(p.loads[0], dtype), 1, 0.002, steps, 0.0, p.vmax, info=info)
    assert np.abs(host(u) - u_ref.ravel()).max() <= _tol(dtype) * np.abs(u_ref).max()
    assert np.abs(host(x) - x_ref).max() <= (1e-9 if dtype == torch.float64 else 2e-5)
    assert host(info)[6] == 0


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("steps", [1, 2, 5])
def test_plane_pcg_few_steps(steps, dtype):
    from paper_2204_06204_amd.grid import PlaneGrid
    from oracle.plane import Grid2D, q4_stiffness
    say(f"plane pcg steps={steps} {dtype}")
    p = synth.plane_config("plane_small")
    og = Grid2D(p.nx, p.ny)
    g = PlaneGrid.from_problem(p, max_rhs=2)
    rho = dev(synth.uniform_density(p.E, 3), dtype)
    s = oracle.simp_scale(host(rho), p.penal, p.rho_min)
    KE = q4_stiffness()
    K = oracle.assemble_K(og, s, p.fixed_mask, KE=KE)
    D = oracle.jacobi_diag(og, s, p.fixed_mask, KE=KE)
    f = np.stack([p.loads[0], -0.5 * np.roll(p.loads[0], -2 * (p.nx + 1))])
    u = torch.zeros(2 * p.ndof, dtype=dtype, device=DEV)
    g.inner_solve(rho, dev(f.ravel(), dtype), u, steps)
    for r, ur in enumerate(host(u).reshape(2, -1)):
        ref, _ = oracle.pcg_ref(lambda v: K @ v, D, f[r], np.zeros(p.ndof), steps)
        assert np.abs(ur - ref).max() <= _tol(dtype) * np.abs(ref).max()
