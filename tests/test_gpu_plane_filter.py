"""The plane grids' Gaussian filter in one launch, at the edges of its 32 x 8
tiles (one tile and less, one element more, more tiles than blocks), with
windows of one, seven and seventeen taps, forward and transposed.
Oracle: the FP64 filter matrix; tolerances of the plane filter's parity test."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle.plane import Grid2D, gaussian_filter_matrix
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,half", [(1, 1, 3), (32, 8, 3), (33, 7, 3), (31, 9, 0), (65, 17, 8), (700, 501, 3)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_plane_filter_tiles(nx, ny, half, dtype):
    from paper_2204_06204_amd.grid import PlaneGrid
    say(f"plane filter tiles {nx}x{ny} half={half} {dtype}")
    og = Grid2D(nx, ny)
    g = PlaneGrid(nx, ny, filter_half=half, filter_sigma=1.4)
    H, Hs = gaussian_filter_matrix(og, half, 1.4)
    x_t = dev(synth.uniform_density(og.E, 7, 0.0, 1.0), dtype)
    x = host(x_t)
    tol = 1e-14 if dtype == torch.float64 else 2e-6
    for tr, ref in ((False, oracle.filter_forward(H, Hs, x)), (True, oracle.filter_transpose(H, Hs, x))):
        out = g.filter(x_t, transpose=tr)
        assert np.abs(host(out) - ref).max() <= tol * (4 if tr else 1)
