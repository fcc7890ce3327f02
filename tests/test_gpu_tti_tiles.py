"""GPU parity of the TTI step at the edges of its tiles (up to 30 words and 32 rows, 256 lanes),
at every radius, against the FP64 oracle.  Gate: one step from identical FP32 inputs, normwise
max error <= 1e-5 as for every step."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.helpers import interior, rel_errors

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("dims", [(120, 8, 3), (121, 9, 2), (3, 33, 12), (29, 37, 1), (64, 17, 9),
                                  (243, 25, 5), (1, 1, 1)], ids=lambda d: "x".join(map(str, d)))
def test_step_at_tile_edges(dims, r):
    import paper_2507_11067_amd as mms
    nx, ny, nz = dims
    grid, nt, n = mms.Grid(nx, ny, nz), 5, 2
    rng = np.random.default_rng(100 * r + nx)

    def field(lo, hi, halo=False):
        a = np.zeros(grid.shape, np.float32)
        v = a if halo else interior(a, grid)
        v[...] = rng.uniform(lo, hi, v.shape).astype(np.float32)
        return a

    c2 = field(0.02, 0.1)
    med = [field(0.05, 0.2), field(0.0, 0.1), field(0.0, 0.8), field(0.0, 6.2)]
    pp, pc, qp, qc = (field(-1, 1, halo=True) for _ in range(4))
    lap = [-2.7, 1.5, -0.2, 0.03, -0.002][:r + 1]
    d1 = [0.8, -0.2, 0.04, -0.004][:r]
    src = (nz - 1, ny // 2, nx // 2)
    f = np.full(nt, 0.3, np.float32)
    dev = lambda a: torch.from_numpy(a).to(DEV)
    traces = torch.zeros((nt, ny, nx), device=DEV)
    w = mms.Wave(grid, dev(c2), lap, nt, 1.0, 3, 0.1, synth.SPONGE_LATERAL_AND_BOTTOM, src, dev(f),
                 traces)
    t = mms.Tti(grid, *(dev(a) for a in med), 0.2, 0.7, d1)
    pn, qn = grid.zeros(DEV).fill_(7.0), grid.zeros(DEV).fill_(7.0)
    w.tti_step(n, t, dev(pp), dev(pc), pn, dev(qp), dev(qc), qn)
    torch.cuda.synchronize()
    ow = oracle.Wave(nx, ny, nz, c2, lap, src, f, nt, 3, 0.1, synth.SPONGE_LATERAL_AND_BOTTOM)
    rp, rq, tr = ow.tti_step(ow.tti(*med, 0.2, 0.7, d1), n, pp, pc, qp, qc)
    for got, ref in ((pn, rp), (qn, rq)):
        g = got.cpu().numpy()
        assert rel_errors(interior(g, grid), interior(ref, grid))[0] <= 1e-5
        interior(g, grid)[...] = 7.0
        assert np.all(g == 7.0)
    np.testing.assert_array_equal(traces[n].cpu().numpy(), tr.astype(np.float32))
