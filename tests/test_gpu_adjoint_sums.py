"""Bits of the log-likelihood's goal gradient.

Betas are added in FP64: weights of +-2^20 on two equal betas cancel, so the
gradient is that of the remaining weight.  Each of the two contributes the same
FP32 value with opposite signs, and n of them add to within n 2^-53 of their
sum of magnitudes: with n = 2 x 3 x 40 terms a goal below 2^20 beta |w| each,
240 x 240 x 2^-53 x 2^20 x 8 < 6e-5 absolute at the very most, while sums in FP32
leave 2^-25 of 2^20 beta per step.

The chosen heading's own unit-vector difference is zero: with a beta so large
that every other heading's probability underflows, the gradient is exactly 0,
also where the step ends close to the goal.
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


def cuda(a):
    return torch.tensor(a, device="cuda")


@pytest.mark.parametrize("K", [4, 8, 12, 16, 32])
def test_cancelling_weights_over_betas(cap, K):
    r = np.random.default_rng(K)
    N, T, G = 3, 40, 5
    th = 2 * np.pi * r.integers(0, K, (N, T)) / K
    steps = 0.06 * np.stack([np.cos(th), np.sin(th)], -1)
    tr = np.concatenate([np.zeros((N, 1, 2)), np.cumsum(steps, 1)], 1)
    tr = (tr + r.uniform(3, 9, (N, 1, 2))).astype(np.float32)
    goals = r.uniform(0, 12, (G, 2)).astype(np.float32)
    lb = np.log(np.array([7.3, 3.1, 7.3, 0.4])).astype(np.float32)
    args = (K, 1.2, 0.05, cuda(tr), cuda(np.full(N, T, np.int32)), cuda(goals), cuda(lb))
    small = r.normal(size=(N, 4, G))
    small[:, [0, 2]] = 0.0
    want, _ = cap.loglik_backward(*args, cuda(small))
    big = small.copy()
    big[:, 0], big[:, 2] = 2.0 ** 20, -(2.0 ** 20)
    got, _ = cap.loglik_backward(*args, cuda(big))
    assert (got - want).abs().max().item() <= 6e-5


@pytest.mark.parametrize("K", [4, 8, 16, 32])
@pytest.mark.parametrize("off", [3e-2, 1e-3, 1e-4])
def test_chosen_heading_has_no_difference_to_itself(cap, K, off):
    r = np.random.default_rng(K)
    N, v, dt = 64, 1.2, 0.05
    th = 2 * np.pi * r.integers(0, K, N) / K
    z = r.uniform(3, 9, (N, 2))
    tr = np.stack([z, z + v * dt * np.stack([np.cos(th), np.sin(th)], 1)], 1).astype(np.float32)
    ph = r.uniform(0, 2 * np.pi, N)
    at = (tr[:, 1] + off * v * dt * np.stack([np.cos(ph), np.sin(ph)], 1)).astype(np.float32)
    # the nearest other heading ends 2 sin(pi / K) steps away: beta times the
    # difference of the two distances is above 130 in base 2
    lb = np.log(np.array([130.0 / (v * dt * (2 * np.sin(np.pi / K) - 2 * off))])).astype(np.float32)
    for n in range(0, N, 16):
        args = (K, v, dt, cuda(tr[n:n + 1]), cuda(np.array([1], np.int32)), cuda(at[n:n + 1]), cuda(lb))
        dg, _ = cap.loglik_backward(*args, torch.ones((1, 1, 1), device="cuda", dtype=torch.float64))
        assert dg.abs().max().item() == 0.0
