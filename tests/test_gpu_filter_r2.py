"""The filter of radius 2 to 3 (two layers of neighbours) at the edges of its
32 x 8 and 16 x 16 tiles and its slabs: shorter than a tile or a stencil, one
past a tile, ragged in every axis.  Oracle: the matrix filter in FP64; the
tolerance is 93 terms' rounding in the result's precision."""
import numpy as np
import pytest
import torch

import synth
from oracle.density_filter import cone_filter_matrix
from oracle.grid import Grid as OGrid
from gpu_util import EPS, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("radius", [2.1, 2.5, 3.0])
@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 1), (3, 2, 5), (16, 17, 4), (17, 8, 9), (33, 9, 5), (64, 7, 37)])
def test_filter_r2(nx, ny, nz, radius, dtype):
    from paper_2204_06204_amd.grid import Grid
    say(f"filter r={radius} {nx}x{ny}x{nz} {dtype}")
    H, Hs = cone_filter_matrix(OGrid(nx, ny, nz), radius)
    g = Grid(nx, ny, nz, filter_radius=radius)
    x = dev(synth.uniform_density(nx * ny * nz, 3, 0.0, 1.0), dtype)
    xh = host(x)
    tol = 100 * EPS[dtype]
    assert np.abs(host(g.filter(x)) - (H @ xh) / Hs).max() <= tol * xh.max()
    ref = H.T @ (xh / Hs)
    assert np.abs(host(g.filter(x, transpose=True)) - ref).max() <= tol * ref.max()
