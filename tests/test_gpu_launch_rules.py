"""The single-human call's launch shapes and the taking of true bounds change no
result: on both sides of every limit the traces of the first particles are the
same, and the counts equal those of a plan of another shape (256 threads x 1
particle and 2 KiB windows, so that nearly every step leaves the LDS), exactly.
Limits at 256 CUs: eight lanes a particle to 16384, four to 32768 (8 headings) or
40960, one beyond, in blocks of 256 (more than 64 controls), 512 (64, or the
shifted draw) or 1024 threads; one speed with a reach beyond the windows in
blocks of 256 up to 64 waves a CU; true bounds never below 16384 particles, where
particles share cells below 131072, always from there on.
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


FLAT = np.array([0.1, 0.5, 2.0, 5.0], np.float32)
SHARP = np.array([30.0, 100.0, 300.0, 600.0], np.float32)      # beta * step up to 72
SHIFTED = np.array([10.0, 100.0, 1000.0, 3000.0], np.float32)


def model(cap, K, S, beta, side):
    r = np.random.default_rng(K + S)
    goals = r.uniform(0.1 * side, 0.9 * side, (5, 2)).astype(np.float32)
    return cap.Model(K, 1.2, 0.1, beta, goals,
                     speeds=np.linspace(0.3, 1.2, S) if S > 1 else None)


@pytest.mark.parametrize("K,S,beta", [(8, 2, FLAT), (8, 8, FLAT), (16, 4, FLAT), (16, 6, FLAT),
                                      (32, 2, FLAT), (32, 3, FLAT), (16, 6, SHIFTED),
                                      (8, 2, SHIFTED)])
def test_lanes_and_blocks_of_several_speeds(cap, K, S, beta):
    m = model(cap, K, S, beta, 10.0)
    bel = torch.full((m.G, m.B), 1.0 / (m.G * m.B), dtype=torch.float64, device="cuda")
    H, n, ref = 7, 16000, None
    for N in (n, 16384, 16385, 32768, 32769, 40960, 40961, 90000, 300000):
        o = cap.predict_occupancy(m, (0.0, 0.0, 0.1, 100, 100), (5.0, 5.0), bel, N, H, seed=2,
                                  human_id=4, cycle=1, trace=True)
        assert torch.all(o["counts"].sum((1, 2)) + o["offgrid"] == N)
        first = (o["trace_k"][:n], o["trace_pair"][:n])
        if ref is None:
            ref = first
        assert torch.equal(first[0], ref[0]) and torch.equal(first[1], ref[1]), N


@pytest.mark.parametrize("K,S,beta,N,H,nx", [
    (16, 1, FLAT, 16383, 60, 200), (16, 1, SHARP, 16384, 60, 200), (8, 1, SHARP, 30000, 60, 200),
    (32, 1, SHIFTED, 30000, 40, 200), (8, 2, SHARP, 30000, 50, 200), (16, 6, SHARP, 20000, 40, 200),
    (16, 1, FLAT, 131071, 40, 200), (16, 1, FLAT, 131072, 40, 200), (16, 1, FLAT, 100000, 80, 700), (12, 1, SHARP, 300000, 80, 700),
    (8, 1, FLAT, 300000, 80, 700), (4, 1, SHARP, 70000, 90, 333), (32, 1, SHARP, 1 << 20, 80, 700),
    (16, 1, SHARP, (1 << 20) + 1, 80, 700)])
def test_counts_do_not_depend_on_shape_or_bounds(cap, K, S, beta, N, H, nx):
    cell = 0.05
    side = nx * cell
    m = model(cap, K, S, beta, side)
    grid = (0.0, 0.0, cell, nx, nx)
    z0 = tuple(float(np.float32(x)) for x in (0.5 * side, 0.45 * side))   # a plan's are FP32
    plan = cap.Plan(K, 1.2, 0.1, 1, ring=1, block_threads=256, particles_per_thread=1,
                    lds_bytes=2048, speeds=m.speeds)
    buf = cap.SlotBuffers.allocate(m, grid, H, 1, probs=False)
    plan.admit(0, 9, m, grid, N, H, z0, buf)
    plan.run(6, 0)
    plan.sync()
    torch.cuda.synchronize()
    o = cap.predict_occupancy(m, grid, z0, buf.belief[0], N, H, seed=6, human_id=9, cycle=0)
    assert torch.equal(o["counts"], buf.counts[0])
    assert torch.equal(o["offgrid"], buf.offgrid[0])
    plan.close()
