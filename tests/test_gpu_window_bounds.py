"""Histogram windows from the particles' bounds, where reach windows outgrow the LDS.

A plan with little LDS (256 and 1024 window words) takes the bounds at every
fourth step at the latest, and its windows go through all three forms; the
single-human call's windows hold every step's reach here.  Counts are whole
numbers and must be equal.  Starts in the middle, at a corner (particles leave the
grid and come back) and outside it; reach of up to three cells a step; horizons
that end on each phase of the four steps.  A grid too large for any LDS is
checked against the oracle.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

BETA = np.array([0.05, 1.0, 20.0], np.float32)
GRID = (0.0, 0.0, 0.1, 60, 50)


@pytest.fixture(scope="module")
def cap():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_01122_amd import capred
    return capred


@pytest.mark.parametrize("lds", [2048, 8192])
@pytest.mark.parametrize("K,S,threads,P", [(12, 1, 256, 1), (16, 1, 512, 2), (8, 1, 1024, 4),
                                           (32, 1, 256, 4), (16, 3, 256, 1), (8, 2, 512, 2)])
@pytest.mark.parametrize("H", [13, 16, 18])
def test_small_windows_count_alike(cap, lds, K, S, threads, P, H):
    starts = [(3.0, 2.5), (0.05, 4.95), (-0.7, 2.0)]
    N = (1, 2049, 5000)
    r = np.random.default_rng(K + H)
    speeds = None if S == 1 else np.linspace(0.4, 1.5, S)
    plan = cap.Plan(K, 1.5, 0.2, 3, ring=2, speeds=speeds, block_threads=threads,
                    particles_per_thread=P, lds_bytes=lds)
    models, bufs = [], []
    for i in range(3):
        goals = r.uniform(0, 6, (4, 2)).astype(np.float32)
        models.append(cap.Model(K, 1.5, 0.2, BETA, goals, speeds=speeds))
        bufs.append(cap.SlotBuffers.allocate(models[i], GRID, H, 2))
        plan.admit(i, 5 + i, models[i], GRID, N[i], H, starts[i], bufs[i])
    moves = [[(x + 0.1, y) for x, y in starts], [(x + 0.2, y - 0.05) for x, y in starts]]
    for c in range(2):
        plan.stage_many([0, 1, 2], moves[c])
        plan.run(9, c)
    plan.sync()
    torch.cuda.synchronize()
    for c in range(2):
        for i in range(3):
            z = np.float32(moves[c][i]).astype(float)
            ref = cap.predict_occupancy(models[i], GRID, z, bufs[i].belief[c], N[i], H, seed=9,
                                        human_id=5 + i, cycle=c)
            torch.cuda.synchronize()
            assert torch.equal(bufs[i].counts[c], ref["counts"])
            assert torch.equal(bufs[i].offgrid[c], ref["offgrid"])
            assert torch.all(ref["counts"].sum((1, 2)) + ref["offgrid"] == N[i])
    plan.close()


@pytest.mark.parametrize("K,S,N", [(16, 1, 3000), (32, 1, 70000), (12, 1, 3000), (16, 2, 3000)])
def test_grid_beyond_the_lds(orc, cap, K, S, N):
    grid, H, z0 = (0.0, 0.0, 0.05, 700, 650), 45, (17.0, 16.0)
    v, dt = 1.5, 0.3                                   # nine cells a step
    goals = np.array([[3.0, 30.0], [34.0, 1.0], [18.0, 17.0]], np.float32)
    speeds = None if S == 1 else np.linspace(0.5, v, S)
    m = cap.Model(K, v, dt, BETA, goals, speeds=speeds)
    bel = np.full(9, 1.0 / 9.0)
    out = cap.predict_occupancy(m, grid, z0, torch.tensor(bel.reshape(3, 3), device="cuda"), N, H,
                                seed=2, human_id=1, cycle=0, trace=True)
    torch.cuda.synchronize()
    kw = dict(K=K, speed=v, dt=dt, beta=BETA, goals=goals, grid=grid, z0=z0, belief=bel, N=N, H=H,
              seed=2, human=1, cycle=0)
    if S > 1:
        kw["speeds"] = speeds
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
