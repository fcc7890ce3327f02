"""The stencil values that a backward pass keeps lie like the other fields of its grid: on a grid of
whole 128-byte rows (Grid.aligned) every interior row starts on a 128-byte line."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_kept_grids_follow_the_layout(monkeypatch):
    import paper_2507_11067_amd as mms
    from paper_2507_11067_amd.autograd import Problem, misfit, propagate
    grid = mms.Grid.aligned(40, 24, 20)
    seen = []
    forward_keep = mms.Wave.forward_keep

    def spy(self, n_begin, n_end, states, kept, stream=None):
        seen.extend(kept)
        return forward_keep(self, n_begin, n_end, states, kept, stream)

    monkeypatch.setattr(mms.Wave, "forward_keep", spy)
    m = grid.zeros(DEV).fill_(2.0).requires_grad_()
    u0, u1 = grid.zeros(DEV), grid.zeros(DEV)
    grid.interior(u1).fill_(0.1)
    prob = Problem(grid, tuple(float(v) for v in synth.LAPLACIAN_R4), 9, 10.0, 1.0,
                   checkpoint_every=4)
    misfit(propagate(m, u0, u1, prob), torch.zeros(9, 24, 40, device=DEV)).backward()
    first = 4 * grid.halo * (grid.sz + grid.sy + 1)     # bytes to the interior's first cell
    assert seen and all(t is None or (t.data_ptr() + first) % 128 == 0 for t in seen)
