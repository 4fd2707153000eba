"""The toy model's tube ratchets around a mean path with a frame that is not a
number, in batches of every launch shape: s and w are not numbers from the first step on,
and the running minima keep their values."""
import numpy as np
import pytest

import oracle as O
from paper_1705_02180_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 5000, 16390])
@pytest.mark.parametrize("K,bad", [(2, 1), (17, 0), (51, 40)])
@pytest.mark.parametrize("axis", [0, 1])
def test_a_nan_frame_shows_in_s_and_w(n, K, bad, axis):
    import torch
    from paper_1705_02180_amd import scps
    t = np.linspace(0.0, 1.0, K)[:, None]
    path = (1 - t) * np.array([[0.0, 5.0]]) + t * np.array([[0.1, 0.2]])
    path[bad, axis] = np.nan
    rng = np.random.default_rng(K)
    xy0 = np.array([[0.0, 4.0]]) + rng.normal(0, 0.5, (n, 2))
    cv0 = np.zeros((n, 8))
    cv0[:, 1] = np.inf
    cv0[:, 5], cv0[:, 6] = 0.25, 0.5
    p = dict(I.funnel_params(), bias_mode=1)
    xy, cv = torch.as_tensor(xy0.copy(), device="cuda"), torch.as_tensor(cv0.copy(), device="cuda")
    scps.funnel_steps(p, xy, cv, 1, mean_path=torch.as_tensor(path, device="cuda"))
    torch.cuda.synchronize()
    got, CV = xy.cpu().numpy(), cv.cpu().numpy()
    want, cvo, _ = O.funnel_steps(p, xy0[:3].copy(), cv0[:3].copy(), 1, mean_path=path)
    assert np.isnan(cvo[:, 3:5]).all() and np.isnan(want).all()
    assert np.isnan(CV[:, 3:5]).all() and np.isnan(got).all()
    assert np.array_equal(CV[:3, 5:7], cvo[:, 5:7]) and np.array_equal(CV[:, 5:7], cv0[:, 5:7])


def test_an_overflowing_distance_gives_no_weights():
    """lambda d beyond the largest float64 for every frame, d itself still finite."""
    import torch
    from paper_1705_02180_amd import scps
    p = dict(I.funnel_params(), bias_mode=1, lam=1e10, kT=0.0)
    path = np.array([[0.0, 5.0], [0.1, 0.2], [0.0, 0.1]])
    xy0 = np.full((2, 2), 1e150)
    cv0 = np.zeros((2, 8))
    cv0[:, 1] = np.inf
    cv0[:, 5], cv0[:, 6] = 0.25, 0.5
    _, cvo, _ = O.funnel_steps(p, xy0.copy(), cv0.copy(), 1, mean_path=path)
    xy, cv = torch.as_tensor(xy0.copy(), device="cuda"), torch.as_tensor(cv0.copy(), device="cuda")
    scps.funnel_steps(p, xy, cv, 1, mean_path=torch.as_tensor(path, device="cuda"))
    torch.cuda.synchronize()
    CV = cv.cpu().numpy()
    assert np.isnan(cvo[:, 3:5]).all() and np.isnan(CV[:, 3:5]).all()
    assert np.array_equal(CV[:, 5:7], cvo[:, 5:7])
