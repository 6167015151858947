"""Edges of the smoothing tiles (64 x 32 cells, every compiled radius and the
radii between), of a plan's skipping of tiles that no particle can have reached,
and of the MPPI rollout's step chunks (48) and block widths (16, 8, 4 waves).

Tolerances as derived for these kernels' parity tests: a smoothed cell is two
sums of 2r + 1 FP32 products and one division, (4 r + 6) 2^-24 relative; MPPI is
FP64 on both sides, 1e-9.
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


@pytest.mark.parametrize("radius", [1, 2, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("ny,nx", [(32, 64), (33, 65), (31, 63), (1, 130), (97, 2)])
def test_smoothing_tile_edges(orc, cap, radius, ny, nx):
    r = np.random.default_rng(radius * 100 + nx)
    counts = r.integers(0, 900, (2, ny, nx)).astype(np.uint32)
    counts[r.random(counts.shape) < 0.5] = 0
    N, sigma = int(counts.sum()) + 3, 0.4 * radius + 0.3
    p = cap.smooth_occupancy(torch.tensor(counts.view(np.int32), device="cuda"), N, sigma, radius)
    got = p.cpu().numpy().astype(np.float64)
    ref = orc.smooth(counts, N, sigma, radius)
    assert np.all(np.abs(got - ref) <= (4 * radius + 6) * 2.0 ** -24 * ref)
    assert np.array_equal(got == 0, ref == 0)


@pytest.mark.parametrize("radius", [1, 3, 7])
def test_plan_smooths_only_what_can_be_reached(cap, radius):
    """A human that walks (and once jumps) across a wide grid: after every cycle
    the whole probability grid is the smoothed count grid, bit for bit, and the
    union grid equals it."""
    grid, N, H = (0.0, 0.0, 0.05, 300, 150), 700, 6
    m = cap.Model(16, 1.2, 0.05, np.array([0.1, 10.0], np.float32),
                  np.array([[14.0, 7.0], [0.2, 0.3]], np.float32))
    plan = cap.Plan(16, 1.2, 0.05, 1, ring=2, max_smooth_radius=8)
    buf = cap.SlotBuffers.allocate(m, grid, H, 2)
    buf.probs.fill_(7.0)                                   # unknown content
    xy = [(2.0, 2.0), (2.06, 2.0), (2.1, 2.05), (13.9, 7.2), (14.9, 7.4), (0.1, 0.1), (0.1, 7.4)]
    plan.admit(0, 5, m, grid, N, H, xy[0], buf, smooth=(1.0, radius))
    union = torch.full((2, H, 150, 300), 3.0, device="cuda")
    plan.set_union(grid, H, union)
    for c, p in enumerate(xy[1:]):
        plan.stage(0, p)
        plan.run(1, c)
        plan.sync()
        torch.cuda.synchronize()
        want = cap.smooth_occupancy(buf.counts[c % 2].contiguous(), N, 1.0, radius)
        torch.cuda.synchronize()
        assert torch.equal(buf.probs[c % 2], want), c
        assert torch.equal(union[c % 2], want), c
    plan.close()


@pytest.mark.parametrize("N,T", [(1, 1), (63, 47), (65, 48), (64, 49), (130, 97), (16385, 50),
                                 (65537, 3)])
def test_mppi_chunks_and_widths(orc, cap, N, T):
    r = np.random.default_rng(N + T)
    H, grid = 30, (0.0, 0.0, 0.1, 64, 80)
    occ = r.random((H, 80, 64)).astype(np.float32) * 0.12
    z0, goal = np.array([3.0, 3.0, 0.8, 0.6]), np.array([5.0, 6.0, 0.0, 0.0])
    U0 = r.normal(scale=0.1, size=(T, 2))
    delta = r.normal(scale=[0.8, 0.6], size=(T, N, 2))
    kw = dict(dt=0.05, tau=20.0, c_time=0.1, **cap.PAPER_MPPI_COST)
    U = torch.tensor(U0, device="cuda")
    S = cap.mppi_step(z0, goal, U, torch.tensor(delta, device="cuda"),
                      occ=torch.tensor(occ, device="cuda"), grid=grid, **kw).cpu().numpy()
    S_o, U_o, near = orc.mppi(z0=z0, goal=goal, U=U0, delta=delta, occ=occ, grid=grid, **kw)
    assert np.all(near == 0)
    assert np.all(np.abs(S - S_o) <= 1e-9 * np.maximum(1.0, np.abs(S_o)))
    assert np.max(np.abs(U.cpu().numpy() - U_o)) <= 1e-9
