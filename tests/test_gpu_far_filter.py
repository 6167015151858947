"""The far-particle filter of the heading draws and the launch shapes of the
single-human call, at the edges of their rules: K with and without a filter,
goals under the start, within a step, just inside and outside the filter's
limit and far away, sharp and flat beliefs, horizons around the sort's limit,
and particle counts around one wave, one block per CU, and two and four
particles per thread.

A filtered draw is the unfiltered one or nothing, so the bar is the one of every
prediction: each particle's first difference from the oracle lies at a CDF tie
within 1e-6 (oracle.tie_check), per-step counts differ by at most 2 per flagged
particle, and counts plus off-grid particles are N.
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


def check(orc, cap, K, v, dt, beta, goals, grid, z0, belief, N, H, cycle=0):
    m = cap.Model(K, v, dt, beta, goals)
    bel = torch.tensor(belief.reshape(m.G, m.B), device="cuda")
    out = cap.predict_occupancy(m, grid, z0, bel, N, H, seed=5, human_id=3, cycle=cycle, trace=True)
    torch.cuda.synchronize()
    kw = dict(K=K, speed=v, dt=dt, beta=beta, goals=goals, grid=grid, z0=z0,
              belief=belief.reshape(-1), N=N, H=H, seed=5, human=3, cycle=cycle)
    ref = orc.predict(**kw)
    st, first = orc.tie_check(other_pair=out["trace_pair"].cpu().numpy(),
                              other_k=out["trace_k"].cpu().numpy(), window=1e-6, **kw)
    assert np.count_nonzero(st == 2) == 0
    counts = out["counts"].cpu().numpy().view(np.uint32).astype(np.int64)
    off = out["offgrid"].cpu().numpy().view(np.uint32).astype(np.int64)
    for t in range(H):
        flagged = np.count_nonzero((st == 1) & (first <= t + 1))
        d = np.abs(counts[t] - ref["counts"][t]).sum() + abs(off[t] - int(ref["offgrid"][t]))
        assert d <= 2 * flagged, (t, d, flagged)
        assert counts[t].sum() + off[t] == N


BETA = np.array([0.01, 0.3, 3.0, 30.0, 100.0], np.float32)
GRID = (0.0, 0.0, 0.05, 120, 100)


# distances of the goals in steps: on the start, within a step, either side of
# the filter's limit (1 / 0.12 = 8.3 steps), far
@pytest.mark.parametrize("K", [4, 8, 12, 16, 32])
@pytest.mark.parametrize("steps", [(0.0, 0.5), (8.0, 8.7), (3.0, 60.0), (200.0, 900.0)])
def test_goals_around_the_limit(orc, cap, K, steps):
    s = 1.2 * 0.05
    z0 = (3.0, 2.5)
    goals = np.array([[z0[0] + d * s * np.cos(a), z0[1] + d * s * np.sin(a)]
                      for d, a in zip(steps, (0.4, 3.9))], np.float32)
    belief = np.full(2 * BETA.size, 1.0 / (2 * BETA.size))
    check(orc, cap, K, 1.2, 0.05, BETA, goals, GRID, z0, belief, 3000, 26)


@pytest.mark.parametrize("H", [23, 24, 25])
@pytest.mark.parametrize("G,B,zeros", [(1, 1, False), (64, 8, False), (40, 5, True)])
def test_sort_of_the_pairs(orc, cap, H, G, B, zeros):
    """One pair, CAP_MAX_J pairs, and a belief with zero entries (the last ones too)."""
    r = np.random.default_rng(G + H)
    beta = np.exp(r.uniform(np.log(0.05), np.log(50), B)).astype(np.float32)
    goals = r.uniform(0, 5, (G, 2)).astype(np.float32)
    belief = r.gamma(1.0, size=G * B)
    if zeros:
        belief[r.uniform(size=G * B) < 0.5] = 0.0
        belief[-7:] = 0.0
        belief[3] = 1.0
    belief /= belief.sum()
    check(orc, cap, 16, 1.2, 0.02, beta, goals, GRID, (3.0, 2.5), belief, 1500, H, cycle=9)


@pytest.mark.parametrize("N", [1, 63, 64, 65, 16384, 16385, 262144, 262145, 524289])
def test_launch_shapes(orc, cap, N):
    """From one wave to four particles per thread (256 CUs: 16384 is one wave
    per CU, 262144 one full block per CU, 524288 two particles per thread)."""
    goals = np.array([[0.5, 0.5], [5.0, 4.0]], np.float32)
    belief = np.full(10, 0.1)
    check(orc, cap, 8, 1.0, 0.1, BETA, goals, GRID, (3.0, 2.5), belief, N, 3)
