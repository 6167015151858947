"""Log-likelihood and adjoint of more tracks than one grid dimension holds
threads for (2^32 at a block of 256 per track): every track gets the value that it
has in a small call, bit for bit, and the shared gradients are the sums of the
small calls'.  Tolerance of the sums: a thread of the second stage adds n = N / 256
terms below 8 in a row, so it errs by at most n 2^-53 8 n, 256 threads by 8 N n
2^-53 = 1e-3, on either side.
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


@pytest.mark.parametrize("per_track", [False, True])
def test_more_than_2_to_24_tracks(cap, per_track):
    N, K, v, dt = (1 << 24) + 77, 8, 1.2, 0.05
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.rand(s, generator=g, device="cuda")
    z = 3.0 + 6.0 * rnd(N, 2)
    th = (rnd(N) * K).floor() * (2 * np.pi / K)
    tr = torch.stack([z, z + v * dt * torch.stack([th.cos(), th.sin()], 1)], 1).contiguous()
    ln = torch.ones(N, dtype=torch.int32, device="cuda")
    goals = torch.tensor([[4.0, 7.0]], device="cuda")
    lb = (rnd(N, 1) if per_track else torch.zeros(1, device="cuda")).contiguous()
    LL = cap.loglik(K, v, dt, tr, ln, goals, lb)
    dLL = rnd(N, 1, 1).double() + 0.5
    dg, db = cap.loglik_backward(K, v, dt, tr, ln, goals, lb, dLL)
    # the same in calls of 2^20 tracks (one track per block there too)
    sg, sb = torch.zeros_like(dg), torch.zeros(1, dtype=torch.float64, device="cuda")
    for a in range(0, N, 1 << 20):
        s = slice(a, min(N, a + (1 << 20)))
        lb_s = lb[s].contiguous() if per_track else lb
        args = (K, v, dt, tr[s].contiguous(), ln[s].contiguous(), goals, lb_s)
        assert torch.equal(cap.loglik(*args), LL[s]), a
        g1, b1 = cap.loglik_backward(*args, dLL[s].contiguous())
        sg += g1
        if per_track:
            assert torch.equal(b1, db[s]), a
        else:
            sb += b1
    tol = 2 * 8 * N * (N / 256) * 2.0 ** -53
    assert (dg - sg).abs().max().item() <= tol
    if not per_track:
        assert (db - sb).abs().max().item() <= tol
