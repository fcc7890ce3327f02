"""GPU parity of the split-precision box over the range of its values: large and small operands,
amplitudes that change along z, and cells that are not finite, against the FP64 oracle.

Tolerance: the FP16 split keeps 22 bits of both operands, so a product is off by less than 2^-21
of itself; operands far below the largest one of their neighbourhood keep fewer, with an absolute
error of 2^-38 of it.  The neighbourhoods below span less than 2^8, which leaves 2^-30: 1e-5 of
the largest output is the bound that every sweep of this library is held to.
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
@pytest.mark.parametrize("xs,cs", [(1e36, 1e-6), (1e-6, 1e34), (1e-36, 1e6), (1e-30, 1e-6),
                                   (1e30, 1e-36), (1e-20, 1e-16)])
def test_fp16_operands_of_any_magnitude(r, xs, cs):
    """A result that fits FP32 is finite and accurate, however far apart the magnitudes of the
    data and the weights are."""
    import paper_2507_11067_amd as mms
    nx, ny, nz = 37, 21, 11
    grid = mms.Grid(nx, ny, nz)
    x = synth.uniform_grid(400, nx, ny, nz, sy=grid.sy) * np.float32(xs)
    c = synth.box_coeffs(401, r) * np.float32(cs)
    ref = interior(oracle.box(x, nx, ny, nz, r, c), grid)
    got = sweep(x, grid, r, c, "fp16x3s")
    assert np.isfinite(got).all()
    assert rel_errors(got, ref)[0] <= 1e-5


@pytest.mark.parametrize("falling", [True, False], ids=["falling", "rising"])
@pytest.mark.parametrize("r", [1, 2, 3, 4])
def test_fp16_scale_follows_the_planes(r, falling):
    """Amplitudes that change by a factor of 0.66 a plane, on a grid of 256 tiles, whose blocks
    walk all 64 planes: every output plane is as accurate as its own neighbourhood allows."""
    import paper_2507_11067_amd as mms
    nx, ny, nz = 1024, 512 if r >= 3 else 1024, 64
    grid = mms.Grid(nx, ny, nz)
    x = synth.uniform_grid(410, nx, ny, nz, sy=grid.sy)
    z = np.arange(nz + 8) - 4
    x *= (0.66 ** (z if falling else nz - 1 - z)).astype(np.float32)[:, None, None]
    c = synth.box_coeffs(411, r)
    got, ref = sweep(x, grid, r, c, "fp16x3s"), interior(oracle.box(x, nx, ny, nz, r, c), grid)
    errors = [rel_errors(got[k], ref[k])[0] for k in range(nz)]
    assert max(errors) <= 1e-5, errors


def bad_cells(grid, r):
    """Cells at corners of tiles, between chunks, at the grid's faces and in the halo that the
    stencil reads: (z, y, x) and value."""
    nx, ny, nz = grid.nx, grid.ny, grid.nz
    nan, inf = np.float32("nan"), np.float32("inf")
    return [((40, 31, 63), nan), ((90, 32, 64), inf), ((141, 3, 4), -inf), ((200, 20, 33), nan),
            ((261, ny - 1, nx - 1), inf), ((nz - 1, 0, 0), nan), ((-1, 10, 10), nan),
            ((300, -r, 20), inf), ((350, 20, nx + r - 1), nan)]


@pytest.mark.parametrize("prec", ["bf16x3", "fp16x3s", "bf16x1"])
@pytest.mark.parametrize("r", [1, 2, 3, 4])
def test_nonfinite_cells_reach_their_box_only(r, prec):
    """A NaN or Inf cell, or in BF16 a value that rounds to Inf, reaches the (2r+1)^3 outputs
    whose box holds it.  Outputs whose tile's window holds it may be summed in another order (the
    gate of every sweep), all others keep their bits."""
    import paper_2507_11067_amd as mms
    nx, ny, nz = 70, 40, 1500
    grid = mms.Grid(nx, ny, nz)
    x = synth.uniform_grid(420, nx, ny, nz, sy=grid.sy)
    c = synth.box_coeffs(421, r)
    cells = bad_cells(grid, r)
    if prec != "fp16x3s":
        cells.append(((400, 8, 40), np.float32(3.4e38)))
    for (zc, yc, xc), _ in cells:
        x[4 + zc, 4 + yc, 4 + xc] = 0.0
    clean = sweep(x, grid, r, c, prec)
    reach, window = np.zeros(clean.shape, bool), np.zeros(clean.shape, bool)
    for (zc, yc, xc), v in cells:
        x[4 + zc, 4 + yc, 4 + xc] = v
        reach[max(zc - r, 0):zc + r + 1, max(yc - r, 0):yc + r + 1, max(xc - r, 0):xc + r + 1] = True
        window[max(zc - r, 0):zc + r + 1, max(yc - r - 3, 0):yc + r + 4, max(xc - 7, 0):xc + 8] = True
    if r < 4:
        x[4 + 450, 4 + 10, 4 + nx + r] = np.nan     # beyond the stencil's reach
        x[4 + 450, 4 + ny + r, 4 + 10] = np.inf
        window[450 - r:450 + r + 1] = True
    got = sweep(x, grid, r, c, prec)
    assert np.isfinite(clean).all()
    assert np.array_equal(got[~window], clean[~window])
    assert np.max(np.abs(got[~reach].astype(np.float64) - clean[~reach])) <= 1e-5 * np.abs(clean).max()
    assert not np.isfinite(got[reach]).any()
    if prec == "bf16x1":
        # one product of an Inf cell and a weight: Inf with the weight's sign
        w = c.reshape((2 * r + 1,) * 3)[::-1, ::-1, ::-1]
        np.testing.assert_array_equal(got[90 - r:90 + r + 1, 32 - r:32 + r + 1, 64 - r:64 + r + 1]
                                      [:, :, :6], (np.sign(w) * np.inf)[:, :, :6].astype(np.float32))
    else:
        assert np.isnan(got[reach]).all()


def test_nonfinite_field_everywhere():
    """A field of NaN gives NaN everywhere, and a finite one after it is as if it had not been."""
    import paper_2507_11067_amd as mms
    nx, ny, nz, r = 70, 40, 400, 3
    grid = mms.Grid(nx, ny, nz)
    x = synth.uniform_grid(430, nx, ny, nz, sy=grid.sy)
    c = synth.box_coeffs(431, r)
    for prec in ("bf16x3", "fp16x3s", "bf16x1"):
        before = sweep(x, grid, r, c, prec)
        assert np.isnan(sweep(np.full_like(x, np.nan), grid, r, c, prec)).all()
        np.testing.assert_array_equal(sweep(x, grid, r, c, prec), before)
