"""GPU parity of the split-precision box at the edges of its tiles (64 x 32 or 64 x 64
outputs), its steps of 2 or 4 input planes and its running FP16 scale, against the FP64 oracle.

Tolerances: the split keeps 16 (BF16) or 22 (FP16) bits of both operands, so a product is off
by less than 2^-16 or 2^-21 of itself before FP32 accumulation, and the errors of (2r+1)^3
products of either sign add up like a random walk; 1e-5 of the largest output is the bound
that every sweep of this library is held to.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.helpers import interior, rel_errors

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def sweep(x, grid, r, c, prec):
    import paper_2507_11067_amd as mms
    out = grid.zeros(DEV)
    mms.stencil_apply(torch.from_numpy(x).to(DEV), out, grid, "box", r, c, precision=prec)
    torch.cuda.synchronize()
    return interior(out.cpu().numpy(), grid)


@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("size", [(63, 31, 1), (65, 33, 3), (64, 65, 6), (130, 4, 37), (3, 97, 70)],
                         ids=lambda s: "x".join(map(str, s)))
def test_tile_edges(r, size):
    import paper_2507_11067_amd as mms
    nx, ny, nz = size
    grid = mms.Grid(nx, ny, nz)
    x = synth.uniform_grid(300 + r, nx, ny, nz, sy=grid.sy)
    c = synth.box_coeffs(310 + r, r)
    ref = interior(oracle.box(x, nx, ny, nz, r, c), grid)
    for prec, tol in (("bf16x3", 1e-5), ("fp16x3s", 1e-5), ("bf16x1", 2e-2)):
        rmax, _ = rel_errors(sweep(x, grid, r, c, prec), ref)
        assert rmax <= tol, (prec, rmax)


@pytest.mark.parametrize("r", [1, 4])
def test_fp16_scale_follows_growing_planes(r):
    """Amplitudes that grow by 2^2 a plane over 40 planes: the scale has to follow them, and
    every output plane is as accurate as its own neighbourhood allows."""
    import paper_2507_11067_amd as mms
    nx, ny, nz = 40, 35, 40
    grid = mms.Grid(nx, ny, nz)
    x = synth.uniform_grid(320, nx, ny, nz, sy=grid.sy)
    x *= (4.0 ** (np.arange(nz + 8) - 30)).astype(np.float32)[:, None, None]
    c = synth.box_coeffs(321, r)
    got, ref = sweep(x, grid, r, c, "fp16x3s"), interior(oracle.box(x, nx, ny, nz, r, c), grid)
    for z in range(nz):
        assert rel_errors(got[z], ref[z])[0] <= 1e-5, z


def test_nonfinite_cells_stay_local():
    """A NaN cell makes NaN of every output within the radius and of none beyond the 4 x 4 tile
    windows that hold it; halo rows beyond the radius are never read."""
    import paper_2507_11067_amd as mms
    nx, ny, nz, r = 70, 40, 30, 2
    grid = mms.Grid(nx, ny, nz, halo=8)
    x = synth.uniform_grid(330, nx, ny, nz, halo=8, sy=grid.sy)
    x[:, :8 - r] = x[:, 8 + ny + r:] = np.nan
    c = synth.box_coeffs(331, r)
    clean = {p: sweep(x, grid, r, c, p) for p in ("bf16x3", "fp16x3s")}
    z, y, xx = 15, 20, 33
    x[8 + z, 8 + y, 8 + xx] = np.nan
    near = np.zeros((nz, ny, nx), bool)
    near[z - r:z + r + 1, y - r - 3:y + r + 4, xx - 7:xx + 8] = True
    for p, ref in clean.items():
        assert np.isfinite(ref).all()
        got = sweep(x, grid, r, c, p)
        assert np.isnan(got[z - r:z + r + 1, y - r:y + r + 1, xx - r:xx + r + 1]).all()
        assert np.array_equal(got[~near], ref[~near])
