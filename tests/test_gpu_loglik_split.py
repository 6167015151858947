"""Log-likelihood and adjoint at the edges of their work split: goals around a
slice (21, 22, 64), tracks with and without a block per CU, steps around a wave's
chunk and around the buffer of recovered controls (1024), empty tracks, motionless
steps, one track and one step, K with and without a compiled kernel, shared and
per-track beta, and goals that a step lands on exactly (the unit vector of a zero
distance counts as 0).

Tolerance: the library's bars, |LL_gpu - LL_oracle| <= 1e-5 max(1, |LL_oracle|)
and gradients within 1e-5 of their norm.
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


def walks(N, T, K, v, dt, seed):
    r = np.random.default_rng(seed)
    th = 2 * np.pi * r.integers(0, K, (N, T)) / K
    steps = v * dt * np.stack([np.cos(th), np.sin(th)], -1)
    steps[:, T // 2:T // 2 + 1] = 0.0                       # one motionless step
    tr = np.concatenate([np.zeros((N, 1, 2)), np.cumsum(steps, 1)], 1)
    return (tr + r.uniform(3, 9, (N, 1, 2))).astype(np.float32)


def check(orc, cap, K, v, dt, tr, lengths, goals, lb, seed):
    t = lambda a: torch.tensor(a, device="cuda")
    per = lb.ndim == 2
    args = (K, v, dt, t(tr), t(lengths), t(goals), t(lb))
    LL = cap.loglik(*args).cpu().numpy()
    dLL = np.random.default_rng(seed).normal(size=LL.shape)
    dg, db = (x.cpu().numpy() for x in cap.loglik_backward(*args, t(dLL)))
    kw = dict(K=K, speed=v, dt=dt, tracks=tr, lengths=lengths, goals=goals.astype(np.float64),
              log_beta=lb.astype(np.float64), per_track_beta=per)
    LL_o = orc.loglik(**kw)
    dg_o, db_o = orc.loglik_grad(dLL=dLL, **kw)
    assert np.all(np.abs(LL - LL_o) <= 1e-5 * np.maximum(1.0, np.abs(LL_o)))
    assert np.linalg.norm(dg - dg_o) <= 1e-5 * np.linalg.norm(dg_o)
    assert np.linalg.norm(db - db_o) <= 1e-5 * np.linalg.norm(db_o)


# (N, T, K, G, B, per-track beta)
SIZES = [(1, 1, 8, 1, 1, False), (3, 64, 16, 1, 4, True), (5, 65, 32, 3, 9, False),
         (300, 9, 4, 21, 5, False), (300, 7, 16, 22, 5, True), (40, 31, 32, 64, 8, False),
         (17, 40, 6, 64, 16, True), (260, 25, 32, 8, 9, False), (2, 1024, 8, 8, 3, False),
         (2, 1025, 32, 5, 3, True), (1, 2100, 12, 2, 2, False)]


@pytest.mark.parametrize("N,T,K,G,B,per", SIZES)
def test_split_edges(orc, cap, N, T, K, G, B, per):
    r = np.random.default_rng(N + 13 * T + G)
    tr = walks(N, T, K, 1.2, 0.05, seed=T + K)
    lengths = r.integers(0, T + 1, N).astype(np.int32)
    lengths[0] = T
    goals = r.uniform(0, 12, (G, 2)).astype(np.float32)
    lb = r.uniform(np.log(0.1), np.log(50), (N, B) if per else B).astype(np.float32)
    check(orc, cap, K, 1.2, 0.05, tr, lengths, goals, lb, seed=G)


@pytest.mark.parametrize("K", [4, 6])
def test_steps_onto_a_goal(orc, cap, K):
    """Half-metre steps on a grid whose points FP32 holds exactly (the first of
    K headings points along x, another back): from, through and onto the goals."""
    x = np.array([0.0, 0.5, 1.0, 1.5, 1.0, 0.5, 0.0])
    tr = np.stack([np.stack([1.0 + x, np.full(7, 2.0)], 1)] * 2).astype(np.float32)
    goals = np.array([[1.5, 2.0], [2.5, 2.0], [1.0, 2.0], [4.0, 2.5]], np.float32)
    lb = np.log(np.array([0.3, 2.0, 8.0])).astype(np.float32)
    check(orc, cap, K, 1.0, 0.5, tr, np.array([6, 3], np.int32), goals, lb, seed=2)
