"""Coefficients reach the library by value, whatever holds them and however it is laid out, and
sweeps run on the current stream."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_every_form_of_coefficients_gives_the_same_sweep():
    import paper_2507_11067_amd as mms
    grid = mms.Grid(33, 21, 17)
    x = torch.from_numpy(synth.uniform_grid(1, 33, 21, 17, sy=grid.sy)).to(DEV)
    c = synth.box_coeffs(5, 1)
    forms = [c, c.tolist(), c.astype(np.float64), np.asfortranarray(c), np.repeat(c, 2, axis=2)[:, :, ::2],
             torch.from_numpy(c), torch.from_numpy(c).to(DEV), c.reshape(-1)]
    outs = [mms.stencil_apply(x, grid.zeros(DEV), grid, "box", 1, f) for f in forms]
    torch.cuda.synchronize()
    for o in outs[1:]:
        assert torch.equal(o, outs[0])
    with pytest.raises(mms.MmsError):
        mms.stencil_apply(x, grid.zeros(DEV), grid, "box", 1, c[:0])
    with pytest.raises(ValueError):
        mms.stencil_apply(x, grid.zeros(DEV), grid, "box", 1, c.astype(">f4"))


def test_sweep_is_ordered_with_its_stream():
    import paper_2507_11067_amd as mms
    grid = mms.Grid(64, 64, 64)
    x, out, ref = grid.zeros(DEV), grid.zeros(DEV), grid.zeros(DEV)
    c = synth.star_coeffs_laplacian(4)
    y = torch.from_numpy(synth.uniform_grid(2, 64, 64, 64, sy=grid.sy)).to(DEV)
    mms.stencil_apply(y, ref, grid, "star", 4, c)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(20):        # work that the sweep has to wait for
            x.normal_()
        x.copy_(y)
        mms.stencil_apply(x, out, grid, "star", 4, c)
    side.synchronize()
    assert torch.equal(out, ref)
