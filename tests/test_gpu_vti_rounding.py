"""The VTI step's FP32 operations, bit for bit: the direct kernel (small grids), the marching one
and its flat tiles (narrow grids) carry out the same operations in the same order."""
import numpy as np
import pytest
import torch

from tests.helpers import interior

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
f32 = np.float32


def fma(a, b, c):
    """a b + c rounded once: the product is exact in 64 bits of mantissa."""
    return (np.asarray(a).astype(np.longdouble) * np.asarray(b) + c).astype(f32)


@pytest.mark.parametrize("dims,r", [((37, 21, 15), 1), ((37, 21, 15), 2), ((64, 30, 20), 3),
                                    ((64, 30, 20), 4), ((170, 150, 150), 4), ((100, 200, 190), 2)],
                         ids=str)
def test_step_matches_its_operations(dims, r):
    import paper_2507_11067_amd as mms
    nx, ny, nz = dims
    grid, n = mms.Grid(nx, ny, nz), 1
    rng = np.random.default_rng(500 + r)
    hp, hc, vp, vc, c2, fa, fb = (rng.uniform(lo, hi, grid.shape).astype(f32) for lo, hi in
                                  [(-1, 1)] * 4 + [(0.02, 0.1), (1, 1.5), (1, 1.2)])
    lap = np.array([-2.7, 1.5, -0.2, 0.03, -0.002][:r + 1], f32)
    c2s = f32(0.37)
    dev = lambda a: torch.from_numpy(a).to(DEV)
    w = mms.Wave(grid, dev(c2), lap, 3, float(c2s))
    hn, vn = grid.zeros(DEV), grid.zeros(DEV)
    w.vti_step(n, dev(fa), dev(fb), dev(hp), dev(hc), hn, dev(vp), dev(vc), vn)
    torch.cuda.synchronize()
    p = min(nz, 18)      # planes compared
    at = lambda a, z=0, y=0, x=0: a[4 + z:4 + z + p, 4 + y:4 + y + ny, 4 + x:4 + x + nx]
    sxy = np.zeros((p, ny, nx), f32)
    szz = np.zeros((p, ny, nx), f32)
    for k in range(-r, r + 1):
        ck = lap[abs(k)]
        sxy = fma(ck, at(hc, y=k) + at(hc, x=k), sxy)
        szz = fma(ck, at(vc, z=k), szz)
    C2 = c2s * at(c2)
    h = fma(C2, fma(at(fa), sxy, at(fb) * szz), fma(2, at(hc), -at(hp)))
    v = fma(C2, fma(at(fb), sxy, szz), fma(2, at(vc), -at(vp)))
    np.testing.assert_array_equal(interior(hn.cpu().numpy(), grid)[:p], h)
    np.testing.assert_array_equal(interior(vn.cpu().numpy(), grid)[:p], v)
