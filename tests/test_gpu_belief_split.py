"""Belief update spread over lanes and blocks, at the edges of its work split:
the smallest model, control counts around the lane groups (8 and 16) and around
a chunk of the Delta buffer, histories around a chunk of transitions, sizes on
both sides of the one-block limit, skipped (motionless) transitions, and a plan
whose update is shared by several blocks.

Tolerance: the library's bar, |log b_gpu - log b_oracle| <= 1e-5 for every
pair.  The plan and the single-human call run the same policy terms and differ
only in the order of FP64 sums: n additions of terms up to |log b| in size err
by at most n 2^-53 max |log b| < 1e-12 here, 1e-10 allowed.
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


def scene(K, S, G, B, n, seed):
    r = np.random.default_rng(seed)
    speeds = np.linspace(0.25, 1.5, S) if S > 1 else None
    beta = np.exp(r.uniform(np.log(0.05), np.log(50), B)).astype(np.float32)
    goals = r.uniform(0, 10, (G, 2)).astype(np.float32)
    v = speeds[r.integers(0, S, n)] if S > 1 else np.full(n, 1.2)
    th = 2 * np.pi * r.integers(0, K, n) / K
    step = 0.1 * v[:, None] * np.stack([np.cos(th), np.sin(th)], 1)
    if n > 4:
        step[n // 2] = 0.0
    obs = np.concatenate([[[5.0, 5.0]], 5.0 + np.cumsum(step, 0)]).astype(np.float32)
    return speeds, beta, goals, obs


def gpu(cap, K, speeds, beta, goals, obs):
    m = cap.Model(K, 1.2, 0.1, beta, goals, speeds=speeds)
    lb = cap.belief_reset(torch.empty((m.G, m.B), dtype=torch.float64, device="cuda"))
    b = torch.empty_like(lb)
    cap.belief_update(m, torch.tensor(obs, device="cuda"), lb, b)
    return m, lb.cpu().numpy(), b.cpu().numpy()


# (K, S, G, B, n_obs)
SIZES = [(2, 1, 1, 1, 1), (8, 1, 2, 4, 10), (9, 1, 3, 3, 5), (16, 1, 1, 9, 65), (17, 1, 64, 8, 3),
         (32, 1, 32, 16, 2), (32, 4, 9, 5, 64), (32, 4, 8, 1, 9), (16, 6, 21, 5, 1),
         (16, 6, 11, 5, 2), (16, 1, 6, 9, 1), (5, 1, 1, 16, 200), (16, 1, 2, 2, 0)]


@pytest.mark.parametrize("K,S,G,B,n", SIZES)
def test_update_at_the_edges_of_the_split(orc, cap, K, S, G, B, n):
    speeds, beta, goals, obs = scene(K, S, G, B, n, 7 * K + n)
    m, lb, b = gpu(cap, K, speeds, beta, goals, obs)
    kw = {} if speeds is None else {"speeds": speeds}
    ref, _, _ = orc.belief_update(K=K, speed=1.2, dt=0.1, beta=beta, goals=goals, obs=obs, **kw)
    assert np.max(np.abs(lb - ref.reshape(G, B))) <= 1e-5
    assert np.max(np.abs(b - np.exp(lb))) <= 1e-15


def test_plan_shares_the_update_between_blocks(cap):
    """21 goals x 96 controls and 8 new observations: several blocks per human,
    the last one normalises; three cycles, beside a human with one block."""
    humans = [(16, 6, 21, 5), (16, 6, 1, 2), (16, 6, 64, 8)]
    sc = [scene(*h, 24, 50 + i) for i, h in enumerate(humans)]
    grid = (0.0, 0.0, 0.1, 100, 100)
    plan = cap.Plan(16, 0.0, 0.1, len(humans), max_obs=8, ring=2, speeds=sc[0][0])
    bufs = []
    for i, (speeds, beta, goals, obs) in enumerate(sc):
        m = cap.Model(16, 0.0, 0.1, beta, goals, speeds=speeds)
        bufs.append(cap.SlotBuffers.allocate(m, grid, 3, 2))
        plan.admit(i, i, m, grid, 600, 3, obs[0], bufs[i])
    for c in range(3):
        for i, (_, _, _, obs) in enumerate(sc):
            plan.stage(i, obs[1 + 8 * c:9 + 8 * c])
        plan.run(0, c)
    plan.sync()
    for i, (speeds, beta, goals, obs) in enumerate(sc):
        _, lb, _ = gpu(cap, 16, speeds, beta, goals, obs)
        assert np.max(np.abs(bufs[i].log_belief.cpu().numpy() - lb)) <= 1e-10
        got = bufs[i].belief[2 % 2].cpu().numpy()
        assert np.max(np.abs(got - np.exp(bufs[i].log_belief.cpu().numpy()))) <= 1e-15
    plan.close()
