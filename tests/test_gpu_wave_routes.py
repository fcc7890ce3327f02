"""A forward call adds the image terms of several steps together, which leaves every bit of
the image as it is."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


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


@pytest.mark.parametrize("block", [1, 2, 3, 8])
@pytest.mark.parametrize("dims", [(37, 22, 18), (327, 118, 97)], ids=["small", "large"])
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
