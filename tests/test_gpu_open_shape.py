"""Plans whose launch shape is left open: particle counts around a tile's quarter,
half and whole (1024, 2048, 4096; several speeds 1024, 2048), many humans past one
tile per CU, and the largest LDS a caller may name.  Counts are whole numbers and
equal the single-human calls'; the per-human launches of the same plan agree.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

BETA = np.array([0.1, 2.0, 15.0], np.float32)
GRID = (0.0, 0.0, 0.1, 64, 48)


@pytest.fixture(scope="module")
def cap():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_01122_amd import capred
    return capred


@pytest.mark.parametrize("K,S", [(12, 1), (16, 1), (32, 1), (16, 3)])
@pytest.mark.parametrize("N", [(1, 1023, 1025), (2048, 4095, 4097), (3000,) * 40, (70001, 20000)])
@pytest.mark.parametrize("lds", [0, 147456])
def test_open_shape(cap, K, S, N, lds):
    H, n = 9, len(N)
    r = np.random.default_rng(K + n)
    speeds = None if S == 1 else np.linspace(0.4, 1.2, S)
    plan = cap.Plan(K, 1.2, 0.1, n, ring=2, speeds=speeds, lds_bytes=lds)
    models, bufs, z = [], [], []
    for i in range(n):
        models.append(cap.Model(K, 1.2, 0.1, BETA, r.uniform(0, 6, (3, 2)).astype(np.float32),
                                speeds=speeds))
        bufs.append(cap.SlotBuffers.allocate(models[i], GRID, H, 2))
        z.append((float(np.float32(r.uniform(1, 5))), float(np.float32(r.uniform(1, 4)))))
        plan.admit(i, 30 + i, models[i], GRID, N[i], H, z[i], bufs[i])
    plan.stage_many(list(range(n)), z)
    plan.run(4, 0)
    plan.stage_many(list(range(n)), z)
    plan.run_plain(4, 1)
    plan.sync()
    torch.cuda.synchronize()
    for c in range(2):
        for i in range(min(n, 6)):
            ref = cap.predict_occupancy(models[i], GRID, z[i], bufs[i].belief[c], N[i], H, seed=4,
                                        human_id=30 + i, cycle=c)
            torch.cuda.synchronize()
            assert torch.equal(bufs[i].counts[c], ref["counts"])
            assert torch.equal(bufs[i].offgrid[c], ref["offgrid"])
    assert plan.stats()[2] == sum(-(-v // 1024) for v in N)
    plan.close()
