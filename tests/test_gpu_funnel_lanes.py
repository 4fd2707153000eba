"""The toy model's tube ratchets with several lanes per trajectory: every launch
shape gives the bits of one lane per trajectory, and the weights' exponential
keeps its extremes."""
import numpy as np
import pytest

import oracle as O
from paper_1705_02180_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1705_02180_amd import scps
    return scps


def path(K):
    t = np.linspace(0.0, 1.0, K)[:, None]
    return (1 - t) * np.array([[0.0, 5.0]]) + t * np.array([[0.1, 0.2]])


def run(S, K, n, xy0, steps):
    import torch
    cv0 = np.zeros((n, 8))
    cv0[:, 1] = cv0[:, 5] = cv0[:, 6] = np.inf
    xy, cv = torch.as_tensor(xy0[:n].copy(), device="cuda"), torch.as_tensor(cv0, device="cuda")
    S.funnel_steps(dict(I.funnel_params(), bias_mode=1), xy, cv, steps, mean_path=torch.as_tensor(path(K), device="cuda"))
    torch.cuda.synchronize()
    return xy.cpu().numpy(), cv.cpu().numpy()


@pytest.mark.parametrize("K", [2, 15, 16, 17, 51, 128])
def test_lane_counts_give_the_same_bits(S, K):
    """16, 8 and 1 lanes per trajectory (at most 4096, at most 16384, more)."""
    rng = np.random.default_rng(K)
    xy0 = np.array([[0.0, 5.0]]) + rng.normal(0, 1.0, (16390, 2))
    one = run(S, K, 16390, xy0, 20)
    for n in (1, 7, 4096, 4097, 16384):
        got = run(S, K, n, xy0, 20)
        assert np.array_equal(got[0], one[0][:n]) and np.array_equal(got[1], one[1][:n]), n


def test_far_positions_match_the_oracle(S):
    """Frames with no weight next to the nearest one (exponents down to -1e12),
    and a position that is not finite."""
    p = dict(I.funnel_params(), bias_mode=1, kT=0.0)
    xy0 = np.array([[0.0, 5.0], [30.0, -2.0], [0.05, 0.3], [400.0, 300.0], [np.nan, 1.0]])
    K = 51
    got, cv = run_at(S, p, K, xy0)
    cv0 = np.zeros((5, 8))
    cv0[:, 1] = cv0[:, 5] = cv0[:, 6] = np.inf
    want, cvo, _ = O.funnel_steps(p, xy0[:4], cv0[:4], 1, mean_path=path(K))
    np.testing.assert_allclose(got[:4], want, rtol=1e-9, atol=1e-9)
    np.testing.assert_allclose(cv[:4, 3:5], cvo[:, 3:5], rtol=1e-9, atol=1e-9)
    assert np.isnan(got[4]).all()


def run_at(S, p, K, xy0):
    import torch
    cv0 = np.zeros((len(xy0), 8))
    cv0[:, 1] = cv0[:, 5] = cv0[:, 6] = np.inf
    xy, cv = torch.as_tensor(xy0.copy(), device="cuda"), torch.as_tensor(cv0, device="cuda")
    S.funnel_steps(p, xy, cv, 1, mean_path=torch.as_tensor(path(K), device="cuda"))
    torch.cuda.synchronize()
    return xy.cpu().numpy(), cv.cpu().numpy()
