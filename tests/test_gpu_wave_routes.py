"""The wave passes choose between a direct kernel (small grids) and a z-marching one, and a
forward call adds the image terms of several steps together: both choices leave every bit of
the results as it is.

The routes are compared through the grid contract: a small grid whose halo holds the
neighbouring cells of a large one must give the large grid's values on its interior.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
DIRECT_MAX = 7 << 19


def weights(r):
    return [-2.9, 1.6, -0.2, 0.025, -0.0018][:r + 1]


def fields(grid, n, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    out = []
    for _ in range(n):
        t = grid.zeros(DEV)
        t.copy_(torch.rand(grid.shape, generator=g, device=DEV) * 0.2 + 0.1)
        out.append(t)
    return out


def cut(t, big, small, z0, y0, x0):
    s = small.zeros(DEV)
    a = t[z0:z0 + small.shape[0], y0:y0 + small.shape[1], x0:x0 + small.nx + 2 * small.halo]
    s[:, :, :a.shape[2]] = a
    return s


@pytest.mark.parametrize("r", [1, 2, 3, 4])
def test_direct_and_marching_passes_agree_bitwise(r):
    import paper_2507_11067_amd as mms
    big = mms.Grid(327, 118, 97)       # ragged in every direction
    small = mms.Grid(61, 35, 29)
    assert big.points > DIRECT_MAX >= small.points
    z0, y0, x0 = 41, 50, 148           # a word of the big grid is a word of the small one
    c2, a, b, u = fields(big, 4, 10 + r)
    cuts = [cut(t, big, small, z0, y0, x0) for t in (c2, a, b, u)]
    res = []
    for grid, (c, p, q, v) in ((big, (c2, a, b, u)), (small, cuts)):
        w = mms.Wave(grid, c, weights(r), 8)
        un, m0, grad = grid.zeros(DEV), grid.zeros(DEV), torch.zeros(
            (grid.nz, grid.ny, grid.nx), dtype=torch.float64, device=DEV)
        w.step(3, p, q, un)
        w.set_accumulation(torch.zeros((grid.nz, grid.ny, grid.nx), device=DEV), 2)
        # steps 6 and 5 of the adjoint: the gradient's terms mu^7 S(u^6) and mu^6 S(u^5); mu^5
        # reads mu^6 beyond the small grid and is not compared
        m1 = grid.zeros(DEV)
        w.adjoint_mu(6, 5, [m0, m1, q, p], us=[v, q], grad=grad)
        res.append((grid.interior(un), grid.interior(m1), grad))
    torch.cuda.synchronize()
    Z, Y, X = slice(z0, z0 + small.nz), slice(y0, y0 + small.ny), slice(x0, x0 + small.nx)
    for k in range(3):
        assert torch.equal(res[0][k][Z, Y, X], res[1][k]), k


@pytest.mark.parametrize("block", [1, 2, 3, 8])
@pytest.mark.parametrize("dims", [(37, 22, 18), (327, 118, 97)], ids=["direct", "marching"])
def test_image_is_the_same_however_steps_are_called(dims, block):
    import paper_2507_11067_amd as mms
    grid, nt = mms.Grid(*dims), 20
    c2, u0, u1 = fields(grid, 3, 5)
    images = []
    for split in (1, 5, nt - 1):       # steps per call
        w = mms.Wave(grid, c2, weights(4), nt, sponge_width=4, sponge_alpha=0.1, sponge_faces=63)
        image = torch.zeros((grid.nz, grid.ny, grid.nx), dtype=torch.float64, device=DEV)
        w.set_image(image, torch.empty(image.shape, device=DEV), block)
        bufs = [u0.clone(), u1.clone(), grid.zeros(DEV)]
        for n in range(1, nt, split):
            end = min(n + split, nt)
            w.forward(n, end, [bufs[(n - 1 + i) % 3] for i in range(end - n + 2)])
        images.append(image)
    torch.cuda.synchronize()
    assert torch.isfinite(images[0]).all() and images[0].max() > 0
    for i in images[1:]:
        assert torch.equal(images[0], i)
