"""A human's belief does not depend on how its update was split: the batched
cycle (an update shared by several blocks), the per-human launches and the
single-human call add the same policy terms in transition order, so the
posteriors are equal bit for bit, several observations per cycle included.
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


# (K, S, G, B): shares of one goal and of several, one pair per share, chunks of
# one transition (64 goals x 128 controls), lane groups of 8 and of 16
@pytest.mark.parametrize("K,S,G,B", [(16, 1, 16, 1), (16, 6, 21, 5), (16, 6, 5, 1), (32, 4, 64, 8),
                                     (32, 4, 64, 1), (8, 1, 64, 2), (8, 1, 2, 4), (16, 1, 3, 9)])
def test_posteriors_do_not_depend_on_the_split(cap, K, S, G, B):
    r = np.random.default_rng(K + G + B)
    speeds = np.linspace(0.3, 1.5, S) if S > 1 else None
    beta = np.exp(r.uniform(np.log(0.05), np.log(50), B)).astype(np.float32)
    goals = r.uniform(0, 10, (G, 2)).astype(np.float32)
    th = r.uniform(0, 2 * np.pi, 24)
    step = r.uniform(0.02, 0.15, (24, 1)) * np.stack([np.cos(th), np.sin(th)], 1)
    step[9] = 0.0
    obs = np.concatenate([[[5.0, 5.0]], 5.0 + np.cumsum(step, 0)]).astype(np.float32)
    m = cap.Model(K, 1.2, 0.1, beta, goals, speeds=speeds)
    grid, H, N = (0.0, 0.0, 0.1, 100, 100), 2, 300
    counts = [8, 5, 1, 3, 7]
    state = {}
    for plain in (False, True):
        plan = cap.Plan(K, 1.2, 0.1, 1, max_obs=8, ring=2, speeds=speeds)
        buf = cap.SlotBuffers.allocate(m, grid, H, 2)
        plan.admit(0, 3, m, grid, N, H, obs[0], buf)
        at, state[plain] = 1, []
        for c, n in enumerate(counts):
            plan.stage(0, obs[at:at + n])
            at += n
            (plan.run_plain if plain else plan.run)(0, c)
            plan.sync()
            torch.cuda.synchronize()
            state[plain].append((buf.log_belief.clone(), buf.belief[c % 2].clone(),
                                 buf.counts[c % 2].clone()))
        plan.close()
    lb = cap.belief_reset(torch.empty((G, B), dtype=torch.float64, device="cuda"))
    b = torch.empty_like(lb)
    at = 0
    for c, n in enumerate(counts):
        cap.belief_update(m, torch.tensor(obs[at:at + n + 1], device="cuda"), lb, b)
        at += n
        for got in (state[False][c], state[True][c]):
            assert torch.equal(got[0], lb), c
            assert torch.equal(got[1], b), c
        assert torch.equal(state[False][c][2], state[True][c][2]), c
