"""The wave passes and the star choose between a direct kernel (small grids) and a z-marching
one in two tile layouts (rows of lanes, flat tiles for narrow grids), and a forward call adds
the image terms of several steps together: these choices leave every bit of the results as it is
(but for the small star, which adds its terms in another order).

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


def passes(grid, c2, a, b, u, r):
    """A star sweep, a forward step, two adjoint steps with their gradient and a VTI step."""
    import paper_2507_11067_amd as mms
    w = mms.Wave(grid, c2, weights(r), 8)
    un, m0, m1, hn, vn, st = (grid.zeros(DEV) for _ in range(6))
    dense = (grid.nz, grid.ny, grid.nx)
    grad = torch.zeros(dense, dtype=torch.float64, device=DEV)
    c = np.linspace(-1, 1, 3 * (2 * r + 1)).astype(np.float32)
    mms.stencil_apply(a, st, grid, "star", r, c)
    w.step(3, a, b, un)
    w.vti_step(3, u, c2, a, b, hn, b, u, vn)
    w.set_accumulation(torch.zeros(dense, device=DEV), 2)
    # steps 6 and 5 of the adjoint: the gradient's terms mu^7 S(u^6) and mu^6 S(u^5); mu^5 reads
    # mu^6 beyond a cut grid and is not compared
    w.adjoint_mu(6, 5, [m0, m1, b, a], us=[u, b], grad=grad)
    torch.cuda.synchronize()
    return [grid.interior(t) for t in (st, un, hn, vn, m1)] + [grad]


# a grid, a part of it (extents, then its place) and what the two run on
PAIRS = {"marching-direct": ((327, 118, 97), (61, 35, 29), (41, 50, 148)),
         "marching-flat": ((120, 261, 240), (61, 259, 239), (1, 2, 24)),
         "flat-direct": ((43, 301, 293), (17, 40, 33), (120, 201, 8))}


@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("pair", PAIRS)
def test_routes_agree_bitwise(pair, r):
    import paper_2507_11067_amd as mms
    dims, part, (z0, y0, x0) = PAIRS[pair]
    big, small = mms.Grid(*dims), mms.Grid(*part)
    assert big.points > DIRECT_MAX and (small.points > DIRECT_MAX) == pair.endswith("flat")
    f = fields(big, 4, 10 + r)
    res = passes(big, *f, r), passes(small, *(cut(t, big, small, z0, y0, x0) for t in f), r)
    Z, Y, X = slice(z0, z0 + small.nz), slice(y0, y0 + small.ny), slice(x0, x0 + small.nx)
    for k, (p, q) in enumerate(zip(*res)):
        if k == 0 and pair.endswith("direct"):    # the small star adds its terms in another order
            assert (p[Z, Y, X] - q).abs().max() <= 1e-5 * q.abs().max()
        else:
            assert torch.equal(p[Z, Y, X], q), k


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


@pytest.mark.parametrize("block", [1, 2, 8])
@pytest.mark.parametrize("dims", [(37, 22, 18), (327, 118, 97), (43, 301, 293)],
                         ids=["direct", "marching", "flat"])
def test_gradient_from_kept_stencil_values_is_the_same(dims, block):
    """The gradient of 13 adjoint steps from forward levels, and from the stencil values S(u^n)
    that the forward steps kept of all, of some and of one of them."""
    import paper_2507_11067_amd as mms
    grid, nt = mms.Grid(*dims), 14
    c2, u0, u1, d = fields(grid, 4, 7)
    w = mms.Wave(grid, c2, weights(4), nt, sponge_width=4, sponge_alpha=0.1, sponge_faces=63)
    us = [u0, u1] + [grid.zeros(DEV) for _ in range(nt - 1)]
    keep = [grid.zeros(DEV).fill_(float("nan")) for _ in range(nt - 1)]
    plain = [u0, u1] + [grid.zeros(DEV) for _ in range(nt - 1)]
    w.forward(1, nt, plain)
    w.forward_keep(1, nt, us, keep)          # keep[n - 1] = S(u^n)
    dense = (grid.nz, grid.ny, grid.nx)
    part = torch.empty(dense, device=DEV)
    resid = torch.ones((nt, grid.ny, grid.nx), device=DEV)

    def run(kept):
        w.set_accumulation(part, block)
        mus = [d.clone(), grid.zeros(DEV)]
        grad = torch.zeros(dense, dtype=torch.float64, device=DEV)
        w.adjoint_mu_keep(nt - 1, 0, [mus[i % 2] for i in range(nt + 2)],
                          [None if k is not None else u for k, u in zip(kept, us)], kept, resid, grad)
        return [grid.interior(t) for t in mus] + [grad]

    mus = [d.clone(), grid.zeros(DEV)]
    ref = torch.zeros(dense, dtype=torch.float64, device=DEV)
    w.set_accumulation(part, block)
    w.adjoint_mu(nt - 1, 0, [mus[i % 2] for i in range(nt + 2)], us=us, resid=resid, grad=ref)
    ref = [grid.interior(t) for t in mus] + [ref]
    every = [None] + keep
    for kept in (every, [k if i % 5 else None for i, k in enumerate(every)],
                 [k if i == 6 else None for i, k in enumerate(every)], [None] * nt):
        for a, b in zip(run(kept), ref):
            assert torch.isfinite(b).all() and torch.equal(a, b)
    for a, b in zip(us, plain):
        assert torch.equal(a, b)


def passes_of_large_grids(grid, c2, a, b, u, r):
    """One forward step without and with an image, with kept stencil values, and one adjoint step
    with the gradient from kept values and from a forward level."""
    import paper_2507_11067_amd as mms
    dense = (grid.nz, grid.ny, grid.nx)
    image, grad, grad2 = (torch.zeros(dense, dtype=torch.float64, device=DEV) for _ in range(3))
    un, ui, uk, s, m0, m1 = (grid.zeros(DEV) for _ in range(6))
    w = mms.Wave(grid, c2, weights(r), 8)
    w.step(3, a, b, un)
    w.forward_keep(3, 4, [a, b, uk], [s])
    w.adjoint_mu_keep(5, 5, [m0, b, a], [None], [u], grad=grad)
    w.adjoint_mu(5, 5, [m1, b, a], us=[u], grad=grad2)
    w.set_image(image)
    w.step(3, a, b, ui)
    part = torch.ones(dense, device=DEV)
    w.set_accumulation(part, 4)     # step 4 is the second of its block: the partial is read
    grad3 = torch.zeros(dense, dtype=torch.float64, device=DEV)
    w.adjoint_mu(3, 3, [m1, b, a], us=[u], grad=grad3)
    torch.cuda.synchronize()
    return [grid.interior(t) for t in (un, ui, uk, s, m0, m1)] + [image, grad, grad2, grad3, part]


# a grid of at least 13 * 2^20 points and a part of it that an other kernel runs
LARGE = {"direct": ((327, 230, 190), (61, 35, 29), (141, 150, 148)),
         "marching": ((240, 241, 243), (239, 190, 183), (1, 20, 52)),
         "flat": ((97, 384, 381), (61, 379, 300), (16, 2, 24))}


@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("kind", LARGE)
def test_large_grids_agree_bitwise(kind, r):
    import paper_2507_11067_amd as mms
    dims, part, (x0, y0, z0) = LARGE[kind]
    big, small = mms.Grid(*dims), mms.Grid(*part)
    assert big.points >= 13 << 20 and small.points < 13 << 20
    assert (small.points <= DIRECT_MAX) == (kind == "direct")
    f = fields(big, 4, 30 + r)
    res = (passes_of_large_grids(big, *f, r),
           passes_of_large_grids(small, *(cut(t, big, small, z0, y0, x0) for t in f), r))
    Z, Y, X = slice(z0, z0 + small.nz), slice(y0, y0 + small.ny), slice(x0, x0 + small.nx)
    for k, (p, q) in enumerate(zip(*res)):
        assert torch.isfinite(q).all() and torch.equal(p[Z, Y, X], q), k


@pytest.mark.parametrize("nz", [1, 2, 3, 10, 11, 21])
def test_few_planes_agree_bitwise(nz):
    """Blocks of one plane, and of a round of the queue of planes with and without a rest."""
    import paper_2507_11067_amd as mms
    part = mms.Grid(301, 47, nz)
    for fn, dims in ((passes, (1210, 3 + 3672000 // (1210 * nz), nz)),
                     (passes_of_large_grids, (2110, 3 + 13632000 // (2110 * nz), nz))):
        big = mms.Grid(*dims)
        assert big.points > (DIRECT_MAX if fn is passes else 13 << 20)
        f = fields(big, 4, 50 + nz)
        res = fn(big, *f, 4), fn(part, *(cut(t, big, part, 0, 60, 500) for t in f), 4)
        for k, (p, q) in enumerate(zip(*res)):
            if fn is passes and k == 0:       # the small star adds its terms in another order
                continue
            assert torch.equal(p[:, 60:60 + part.ny, 500:500 + part.nx], q), k
