"""The records of several outer iterations in one call, where the filter-step
pass of an iteration writes the solve's part of its own record and completes
the one before: no iteration (n = 1), one and several deferred, with a search
budget of one pass (the projection's status enters a record late), with a
non-finite load (the solve's does), and a grid of one filter tile.  Oracle:
single calls, whose records one launch writes; bitwise, but the volume (the
same sum over other partial groupings) to 1e-12."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import DEV, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,n", [(8, 3, 3, 2), (70, 13, 9, 1), (70, 13, 9, 5)])
@pytest.mark.parametrize("kind", ["plain", "one_pass", "nonfinite"])
def test_records_equal_single_calls(nx, ny, nz, n, kind):
    from paper_2204_06204_amd.grid import Grid
    say(f"outer records {nx}x{ny}x{nz} n={n} {kind}")
    p = synth.cantilever(nx, ny, nz, volfrac=0.3, filter_radius=1.5, outer_iters=n, inner_steps=4, seed=8)
    f = dev(p.loads[0], torch.float32)
    if kind == "nonfinite":
        f[f.nonzero()[0]] = float("nan")
    res = []
    for multi in (False, True):
        g = Grid.from_problem(p)
        if kind == "one_pass":
            g.set_option("proj_passes", 1)
        x = g.project_volume(dev(p.x0, torch.float32), lo=0.0, hi=1.0, vmax=p.vmax)
        u = torch.zeros(p.ndof, dtype=torch.float32, device=DEV)
        info = torch.full((8 * n,), -7.0, dtype=torch.float64, device=DEV)
        a0 = 0.002 if kind == "plain" else 0.5
        if multi:
            g.outer_steps(x, u, f, 1, n, a0, p.inner_steps, 0.0, p.vmax, info=info)
        else:
            for k in range(1, n + 1):
                g.outer_step(x, u, f, k, a0, p.inner_steps, 0.0, p.vmax, info=info[8 * (k - 1):8 * k])
        res.append((host(x).copy(), host(info).reshape(n, 8).copy()))
        g.close()
    (x1, i1), (x2, i2) = res
    assert np.array_equal(x1, x2, equal_nan=True)
    rest = [c for c in range(8) if c != 4]
    assert np.array_equal(i1[:, rest], i2[:, rest], equal_nan=True), (i1, i2)
    np.testing.assert_allclose(i2[:, 4], i1[:, 4], rtol=0.0, atol=1e-12 * p.vmax)
    if kind == "nonfinite":
        assert (i2[:, 6] != 0).all()
