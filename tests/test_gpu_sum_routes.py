"""On large grids the passes that add to an image or gradient run in one of two marching kernels, by
the length of a row and by whether a step adds one term or several: the sums do not depend on it.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("block", [1, 8])
@pytest.mark.parametrize("r", [1, 3, 4])
@pytest.mark.parametrize("dims", [(240, 241, 243), (241, 238, 243), (100, 400, 360)],
                         ids=["whole-words", "odd-rows", "flat"])
def test_image_by_single_steps_and_by_one_call(dims, r, block):
    import paper_2507_11067_amd as mms
    grid, nt = mms.Grid(*dims), 7
    assert grid.points >= 13 << 20
    gen = torch.Generator(device=DEV).manual_seed(60 + r)
    c2, u0, u1 = (torch.rand(grid.shape, generator=gen, device=DEV) * 0.2 + 0.1 for _ in range(3))
    images = []
    for split in (1, 2, nt - 1):       # steps per call
        w = mms.Wave(grid, c2, [-2.9, 1.6, -0.2, 0.025, -0.0018][:r + 1], nt, sponge_width=4,
                     sponge_alpha=0.1, sponge_faces=63)
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
