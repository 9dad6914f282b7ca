"""Fused CG and MINRES steps on grids of 2^21 elements and more that are two
elements wide or two layers thick: tiles made for wide planes leave most of
their threads idle there, and a step then took three to five times as long as
on a cube of as many elements.  The steps are bound by memory, so a grid's
time goes with its nodes; the limit is about twice that.  A solve on each of these
grids is also compared with the same solve under another tile (the tile changes
the order of the partial sums only)."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, host, say

pytestmark = pytest.mark.gpu


def _grid(size):
    from paper_2204_06204_amd.grid import Grid
    nx, ny, nz = size
    mask = np.zeros((nz + 1, ny + 1, nx + 1, 3), np.uint8)
    mask[:, 0, :, :] = 1
    return Grid(nx, ny, nz, fixed_mask=mask.reshape(-1)), mask.reshape(-1)


def _inputs(g, mask, dtype):
    gen = torch.Generator(device=DEV).manual_seed(7)
    free = torch.tensor(mask == 0, device=DEV)
    rho = (0.2 + 0.6 * torch.rand(g.E, generator=gen, device=DEV, dtype=torch.float64)).to(dtype)
    f = ((torch.rand(g.ndof, generator=gen, device=DEV, dtype=torch.float64) - 0.5) * free).to(dtype)
    return rho, f


def _step_ms(g, rho, f, method):
    u = torch.zeros_like(f)

    def run(n):
        g.inner_solve(rho, f, u, n, method=method, omega=1.0)

    def best(n):
        run(n)
        t = float("inf")
        for _ in range(3):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            run(n)
            b.record()
            torch.cuda.synchronize()
            t = min(t, a.elapsed_time(b))
        return t

    return (best(25) - best(5)) / 20


@pytest.mark.parametrize("method", ["pcg", "krylov"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_narrow_grid_step_time(dtype, method):
    ms = {}
    for size in ((130, 130, 130), (2, 1048, 1048)):
        g, mask = _grid(size)
        rho, f = _inputs(g, mask, dtype)
        ms[size] = _step_ms(g, rho, f, method) / g.N
        say(f"{method} {dtype} {size}: {ms[size] * g.N:.4f} ms a step")
        g.close()
    limit = 2.0 if dtype == torch.float64 else 2.5  # FP32 times of a grid vary more from process to process
    assert ms[2, 1048, 1048] <= limit * ms[130, 130, 130]


@pytest.mark.parametrize("size", [(2, 1048, 1048), (1048, 1048, 2), (8, 524, 524), (20, 331, 331)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_narrow_grid_solve(dtype, size):
    say(f"narrow {size} {dtype}")
    g, mask = _grid(size)
    rho, f = _inputs(g, mask, dtype)
    out = []
    for tile in (0, 15 | 15 << 8):  # slab depth left to the cost model
        g.set_option("cgf_tile", tile)
        u = torch.zeros_like(f)
        info = torch.zeros(8, dtype=torch.float64, device=DEV)
        g.inner_solve(rho, f, u, 5, info=info)
        assert host(info)[3] == 5 and host(info)[4] == 0
        out.append(host(u))
    # partial sums in another order: a few roundings of the step's scalars
    tol = 1e-12 if dtype == torch.float64 else 1e-5
    assert np.abs(out[0] - out[1]).max() <= tol * np.abs(out[1]).max()
    g.close()
