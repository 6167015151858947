"""The filter of far particles changes no heading: one speed (filtered) against
two speeds of which the mask allows the first only (draw_control and
wide_control have no filter and evaluate that speed by the same operations).
Traces, pairs, counts and off-grid counts are equal, exactly, over 10^7 draws a
case: goals from just outside the filter's limit (8.3 steps) to far away, flat
beliefs to the sharpest that the unshifted exponent takes, fine lattice steps to
the coarsest that the filter takes.
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


# N: several lanes a particle in the unfiltered call, and one
@pytest.mark.parametrize("N,H", [(1 << 14, 60), (1 << 18, 40)])
@pytest.mark.parametrize("step", [0.06, 0.0034])    # 78600 and 4456 lattice units
@pytest.mark.parametrize("K", [8, 16, 32])
def test_filtered_headings_are_the_unfiltered_ones(cap, K, step, N, H):
    r = np.random.default_rng(K + H)
    dt, grid, z0 = 0.05, (0.0, 0.0, 0.05, 130, 120), (3.0, 2.5)
    v = step / dt
    d = step * np.array([8.5, 9.0, 11.0, 16.0, 30.0, 70.0, 150.0, 800.0])
    a = r.uniform(0, 2 * np.pi, d.size)
    goals = np.stack([z0[0] + d * np.cos(a), z0[1] + d * np.sin(a)], 1).astype(np.float32)
    beta = (np.array([0.1, 2.0, 10.0, 30.0, 56.0, 79.0]) / step).astype(np.float32)
    G, B = d.size, beta.size
    belief = torch.full((G, B), 1.0 / (G * B), dtype=torch.float64, device="cuda")
    one = cap.Model(K, v, dt, beta, goals)
    two = cap.Model(K, v, dt, beta, goals, speeds=np.array([v, 0.5 * v]), speed_mask=1)
    f = cap.predict_occupancy(one, grid, z0, belief, N, H, seed=11, human_id=2, trace=True)
    g = cap.predict_occupancy(two, grid, z0, belief, N, H, seed=11, human_id=2, trace=True)
    for k in ("trace_pair", "trace_k", "counts", "offgrid"):
        assert torch.equal(f[k], g[k]), k
