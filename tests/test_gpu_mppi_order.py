"""MPPI: a sample's cost is the same bits in any batch (the launch's waves per
block follow from the batch size), and the weights hold for every accepted
temperature, down to those whose reciprocal is not finite.
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


def costs(cap, delta, T, tau=20.0):
    r = np.random.default_rng(5)
    grid = (0.0, 0.0, 0.1, 64, 80)
    occ = torch.tensor(r.random((30, 80, 64)).astype(np.float32) * 0.12, device="cuda")
    U = torch.tensor(r.normal(scale=0.1, size=(T, 2)), device="cuda")
    U0 = U.clone()
    S = cap.mppi_step((3.0, 3.0, 0.8, 0.6), (5.0, 6.0, 0.0, 0.0), U, delta, dt=0.05, tau=tau,
                      c_time=0.1, occ=occ, grid=grid, **cap.PAPER_MPPI_COST)
    return S, U, U0


@pytest.mark.parametrize("T", [1, 5, 48, 97])
def test_cost_does_not_depend_on_the_batch(cap, T):
    g = torch.Generator(device="cuda").manual_seed(T)
    delta = torch.randn((T, 70000, 2), generator=g, device="cuda", dtype=torch.float64)
    few, _, _ = costs(cap, delta[:, :100].contiguous(), T)
    for n in (16385, 70000):   # 16 waves a block up to 16384 samples, 8 to 65536, then 4
        many, _, _ = costs(cap, delta[:, :n].contiguous(), T)
        assert torch.equal(many[:100], few), n


@pytest.mark.parametrize("tau", [5e-324, 1e-309, 1e-300, 1e300])
def test_extreme_temperatures(cap, tau):
    T, N = 7, 300
    g = torch.Generator(device="cuda").manual_seed(1)
    delta = torch.randn((T, N, 2), generator=g, device="cuda", dtype=torch.float64)
    S, U, U0 = costs(cap, delta, T, tau)
    if tau < 1.0:     # only the cheapest sample has a weight
        want = U0 + delta[:, int(S.argmin())]
        assert torch.equal(U, want)
    else:             # equal weights; 300 additions of terms near 1
        want = U0 + delta.mean(1)
        assert torch.max((U - want).abs()).item() < 300 * 2.0 ** -53 * 4


def test_infinite_and_undefined_costs(cap):
    """A sample whose cost is infinite has weight 0; a NaN cost makes the controls NaN."""
    T, N = 5, 200
    g = torch.Generator(device="cuda").manual_seed(2)
    delta = torch.randn((T, N, 2), generator=g, device="cuda", dtype=torch.float64)
    some = delta.clone()
    some[1, 100:, 0] = 1e200            # cost overflows
    S, U, U0 = costs(cap, some, T)
    assert torch.isinf(S[100:]).all() and torch.isfinite(S[:100]).all()
    w = torch.exp((S[:100].min() - S[:100]) / 20.0)
    d = delta[:, :100]
    want = U0 + (w[None, :, None] * d).sum(1) / w.sum()
    keep = torch.tensor([0, 2, 3, 4], device="cuda")
    assert torch.max((U - want)[keep].abs()).item() < 100 * 2.0 ** -53 * 8
    some[1, 150, 0] = float("nan")
    _, U, _ = costs(cap, some, T)
    assert torch.isnan(U).all()
