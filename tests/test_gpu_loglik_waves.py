"""Log-likelihood and adjoint for every number of waves that a block can have: one
to four for tracks of few chunks of steps (even and uneven splits, the 768-thread
adjoint of 32 headings included), eight, twelve and sixteen while the tracks do
not fill the device.  Tolerances: the library's bars, as in
test_gpu_loglik_split.py.
"""
import numpy as np
import pytest

from test_gpu_loglik_split import cap, check, walks  # noqa: F401

pytestmark = pytest.mark.gpu


# (N, T, K, G, B): with one goal a chunk is 64 steps, with five 12
@pytest.mark.parametrize("N,T,K,G,B", [
    (2000, 5, 32, 1, 1), (1500, 65, 16, 1, 3), (1100, 129, 8, 1, 2), (1030, 49, 32, 5, 4),
    (1030, 60, 12, 5, 9), (1030, 100, 32, 5, 9), (600, 200, 8, 5, 2), (500, 100, 32, 5, 16),
    (250, 120, 32, 5, 16), (250, 200, 16, 5, 3), (129, 9, 24, 2, 16)])
def test_waves_per_block(orc, cap, N, T, K, G, B):  # noqa: F811
    r = np.random.default_rng(N + T)
    tr = walks(N, T, K, 1.2, 0.05, seed=T + K)
    lengths = r.integers(0, T + 1, N).astype(np.int32)
    lengths[:2] = T
    goals = r.uniform(0, 12, (G, 2)).astype(np.float32)
    lb = r.uniform(np.log(0.1), np.log(50), B).astype(np.float32)
    check(orc, cap, K, 1.2, 0.05, tr, lengths, goals, lb, seed=G)
