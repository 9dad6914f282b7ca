"""CG on a grid of 2^19 elements and more, where the fused steps update the
iterate in pairs: two, three and four steps have one fused step (a single
update), two (a pair) and three (a pair and a single one).  Oracle and
tolerances: textbook Jacobi-PCG in FP64 by the element loop, those of the PCG
tests on small grids."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle.grid import Grid as OGrid
from gpu_util import DEV, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_pcg_pairs(dtype):
    from paper_2204_06204_amd.grid import Grid
    say(f"pcg pairs {dtype}")
    p = synth.cantilever(131, 67, 61, volfrac=0.3, filter_radius=1.5, outer_iters=1, inner_steps=4, seed=4)
    og = OGrid(p.nx, p.ny, p.nz)
    assert p.E >= 1 << 19
    g = Grid.from_problem(p)
    rho = dev(synth.uniform_density(p.E, 3), dtype)
    s = oracle.simp_scale(host(rho), p.penal, p.rho_min)
    D = oracle.jacobi_diag(og, s, p.fixed_mask)
    rng = np.random.default_rng(5)
    u0 = dev(np.where(p.fixed_mask == 0, 0.1 * rng.standard_normal(p.ndof), 0.0), dtype)
    f = dev(p.loads[0], dtype)
    tol = 1e-10 if dtype == torch.float64 else 2e-4
    for steps in (2, 3, 4):
        u = u0.clone()
        info = torch.zeros(8, dtype=torch.float64, device=DEV)
        g.inner_solve(rho, f, u, steps, info=info)
        ref, res = oracle.pcg_ref(lambda v: oracle.apply_K(og, s, v, p.fixed_mask), D, p.loads[0], host(u0), steps)
        assert np.abs(host(u) - ref).max() <= tol * np.abs(ref).max()
        inf = host(info)
        assert inf[3] == steps and inf[4] == 0
        assert abs(inf[0] - np.linalg.norm(res)) <= (1e-8 if dtype == torch.float64 else 1e-2) * np.linalg.norm(res)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_krylov_pairs(dtype):
    """Degrees 1 to 4: one fused pass, and with two, three and four passes a
    single direction, a pair, and a pair and a single one.  Tolerances of the
    Krylov parity tests on small grids."""
    from paper_2204_06204_amd.grid import Grid
    say(f"krylov pairs {dtype}")
    p = synth.cantilever(131, 67, 61, volfrac=0.3, filter_radius=1.5, outer_iters=1, inner_steps=4, seed=4)
    og = OGrid(p.nx, p.ny, p.nz)
    g = Grid.from_problem(p)
    rho = dev(synth.uniform_density(p.E, 3, 0.3, 1.0), dtype)
    s = oracle.simp_scale(host(rho), p.penal, p.rho_min)
    rng = np.random.default_rng(6)
    u0 = dev(np.where(p.fixed_mask == 0, 0.1 * rng.standard_normal(p.ndof), 0.0), dtype)
    f = dev(p.loads[0], dtype)
    tol = 1e-9 if dtype == torch.float64 else 3e-4
    for deg in (1, 2, 3, 4):
        u = u0.clone()
        g.inner_solve(rho, f, u, deg, method="krylov", omega=1.0)
        ref, _ = oracle.krylov_step_ref(lambda v: oracle.apply_K(og, s, v, p.fixed_mask), p.loads[0], host(u0), deg)
        assert np.abs(host(u) - ref).max() <= tol * np.abs(ref - host(u0)).max(), deg
