"""Multi-speed draws by 8, 4 and 1 lanes per particle are the same draws.

A particle's stream depends on its index alone, so the first particles of a call
draw the same controls whatever the particle count, which chooses the lanes: on
256 CUs 8 lanes up to 16384 particles (K >= 16), 4 up to 65536 (K >= 8), 1 beyond.
Compared bit for bit (controls, pairs), for K and S at their ends, masks with
the first, last, middle and all but one speed excluded, near and far goals; and a
plan whose cycle crosses the particle count from which one lane takes a particle.
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


GRID = (0.0, 0.0, 0.1, 60, 70)
BETA = np.array([0.05, 1.0, 10.0, 60.0], np.float32)


def model(cap, K, S, mask, seed):
    r = np.random.default_rng(seed)
    goals = r.uniform(0, 6, (5, 2)).astype(np.float32)
    goals[0] = (3.05, 3.02)                      # within a step of the start
    return cap.Model(K, 0.0, 0.2, BETA, goals, speeds=np.linspace(0.2, 1.5, S), speed_mask=mask)


@pytest.mark.parametrize("K,S,mask", [(4, 2, 0), (8, 2, 0), (8, 8, 0b10110110), (16, 6, 0),
                                      (16, 6, 0b111110), (16, 6, 0b011111), (16, 6, 0b001000),
                                      (16, 8, 0), (32, 4, 0), (32, 3, 0b101), (32, 2, 0b01)])
def test_lanes_per_particle_draw_alike(cap, K, S, mask):
    m = model(cap, K, S, mask, K + S)
    bel = torch.full((m.G, m.B), 1.0 / (m.G * m.B), dtype=torch.float64, device="cuda")
    H, n = 7, 16383
    out = [cap.predict_occupancy(m, GRID, (3.0, 3.0), bel, N, H, seed=11, human_id=2, cycle=4,
                                 trace=True) for N in (n, 16384, 16385, 65536, 65537)]
    torch.cuda.synchronize()
    for o in out[1:]:
        assert torch.equal(o["trace_pair"][:n], out[0]["trace_pair"])
        assert torch.equal(o["trace_k"][:n], out[0]["trace_k"])
    assert torch.equal(out[2]["trace_k"], out[3]["trace_k"][:16385])
    for o, N in zip(out, (n, 16384, 16385, 65536, 65537)):
        assert torch.all(o["counts"].sum((1, 2)) + o["offgrid"] == N)


@pytest.mark.parametrize("K,P,threads", [(8, 2, 256), (16, 1, 0), (16, 4, 512), (32, 1, 1024)])
@pytest.mark.parametrize("extra", [0, 1])
def test_plan_around_the_wide_limit(cap, K, P, threads, extra):
    """Two humans of 65536 particles together (four lanes each) and one more
    particle (one lane each): both equal the single-human calls bit for bit."""
    N, H, S = (5000, 60536 + extra), 4, 4
    plan = cap.Plan(K, 0.0, 0.2, 2, ring=2, speeds=np.linspace(0.2, 1.5, S),
                    block_threads=threads, particles_per_thread=P)
    bufs = []
    for i in range(2):
        m = model(cap, K, S, 0, 3 + i)
        bufs.append(cap.SlotBuffers.allocate(m, GRID, H, 2))
        plan.admit(i, 7 + i, m, GRID, N[i], H, (3.0, 3.0), bufs[i])
    for c, p in enumerate([(3.02, 3.0), (3.1, 3.05)]):
        plan.stage_many([0, 1], [p, p])
        plan.run(3, c)
    plan.sync()
    torch.cuda.synchronize()
    for i in range(2):
        for c, p in enumerate([(3.02, 3.0), (3.1, 3.05)]):
            p32 = np.float32(p).astype(float)
            ref = cap.predict_occupancy(model(cap, K, S, 0, 3 + i), GRID, p32,
                                        bufs[i].belief[c], N[i], H, seed=3, human_id=7 + i, cycle=c)
            torch.cuda.synchronize()
            assert torch.equal(bufs[i].counts[c], ref["counts"])
            assert torch.equal(bufs[i].offgrid[c], ref["offgrid"])
    plan.close()
