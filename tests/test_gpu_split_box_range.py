"""GPU parity of the split-precision box over the range of its values: large and small operands,
and amplitudes that change along z, against the FP64 oracle.

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
