"""GPU parity on grids that are long in z, against the FP64 oracle, every plane compared.  The z chunks
of a launch come from the number of tile columns, so a grid of few columns and 2600 planes gives
each block a chunk of several planes (box FP32: 31 at radius 1, 11 above; split boxes: 21 at radii
1 and 2, 41 at 3 and 4; TTI: 11), with a shorter last one: what a small cube, whose chunks are one
plane long, does not reach.  Gates: 1e-5 normwise as for every sweep and step, 2e-2 for BF16X1."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.helpers import interior, rel_errors

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NZ = 2600


@pytest.mark.parametrize("r", [1, 2, 3, 4])
def test_box_chunks(r):
    import paper_2507_11067_amd as mms
    nx, ny = 70, 40
    grid = mms.Grid(nx, ny, NZ)
    x = synth.uniform_grid(600 + r, nx, ny, NZ, sy=grid.sy)
    c = synth.box_coeffs(610 + r, r)
    ref = interior(oracle.box(x, nx, ny, NZ, r, c), grid)
    xd = torch.from_numpy(x).to(DEV)
    for prec, tol in (("fp32", 1e-5), ("bf16x3", 1e-5), ("fp16x3s", 1e-5), ("bf16x1", 2e-2)):
        out = grid.zeros(DEV).fill_(7.0)
        mms.stencil_apply(xd, out, grid, "box", r, c, precision=prec)
        got = out.cpu().numpy()
        assert rel_errors(interior(got, grid), ref)[0] <= tol, prec
        interior(got, grid)[...] = 7.0
        assert np.all(got == 7.0), prec


@pytest.mark.parametrize("r", [1, 2, 3, 4])
def test_tti_chunks(r):
    import paper_2507_11067_amd as mms
    nx, ny, nt, n = 33, 9, 5, 2
    grid = mms.Grid(nx, ny, NZ)
    rng = np.random.default_rng(620 + r)

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
    src = (NZ - 1, ny // 2, nx // 2)
    f = np.full(nt, 0.3, np.float32)
    dev = lambda a: torch.from_numpy(a).to(DEV)
    traces = torch.zeros((nt, ny, nx), device=DEV)
    w = mms.Wave(grid, dev(c2), lap, nt, 1.0, 3, 0.1, synth.SPONGE_LATERAL_AND_BOTTOM, src, dev(f),
                 traces)
    t = mms.Tti(grid, *(dev(a) for a in med), 0.2, 0.7, d1)
    pn, qn = dev(pp), dev(qp)      # in place: next = prev
    w.tti_step(n, t, pn, dev(pc), pn, qn, dev(qc), qn)
    torch.cuda.synchronize()
    ow = oracle.Wave(nx, ny, NZ, c2, lap, src, f, nt, 3, 0.1, synth.SPONGE_LATERAL_AND_BOTTOM)
    rp, rq, tr = ow.tti_step(ow.tti(*med, 0.2, 0.7, d1), n, pp, pc, qp, qc)
    for got, ref, prev in ((pn, rp, pp), (qn, rq, qp)):
        g = got.cpu().numpy()
        assert rel_errors(interior(g, grid), interior(ref, grid))[0] <= 1e-5
        interior(g, grid)[...] = interior(prev, grid)
        np.testing.assert_array_equal(g, prev)
    np.testing.assert_array_equal(traces[n].cpu().numpy(), tr.astype(np.float32))
