"""A plan writes a smoothed slot's whole probability grid each cycle: what the
caller wrote into its buffer between two cycles (an in-place transform, say) is
gone after the next one, also where no particle can have come.  Exact: the grid
equals cap_smooth_occupancy of the counts, bit for bit.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cap():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_01122_amd import capred
    return capred


@pytest.mark.parametrize("plain", [False, True])
@pytest.mark.parametrize("nx,ny", [(300, 150), (65, 33), (64, 257)])
def test_smoothed_grids_are_written_whole(cap, nx, ny, plain):
    grid, N, H, radius = (0.0, 0.0, 0.05, nx, ny), 500, 4, 2
    m = cap.Model(16, 1.2, 0.05, np.array([0.1, 10.0], np.float32),
                  np.array([[1.0, 1.0], [0.2, 0.3]], np.float32))
    plan = cap.Plan(16, 1.2, 0.05, 1, ring=2, max_smooth_radius=8)
    buf = cap.SlotBuffers.allocate(m, grid, H, 2)
    plan.admit(0, 5, m, grid, N, H, (0.8, 0.8), buf, smooth=(1.0, radius))
    for c in range(5):
        plan.stage(0, (0.8 + 0.01 * c, 0.8))
        (plan.run_plain if plain else plan.run)(1, c)
        plan.sync()
        torch.cuda.synchronize()
        want = cap.smooth_occupancy(buf.counts[c % 2].contiguous(), N, 1.0, radius)
        assert torch.equal(buf.probs[c % 2], want), c
        buf.probs[c % 2].mul_(0.5).add_(0.25)
        torch.cuda.synchronize()
    plan.close()
