"""Toy-model batches on both sides of every line at which the lanes per
trajectory change with the frames of the mean path: the first trajectories have
the bits of a batch that runs one lane each."""
import numpy as np
import pytest

from paper_1705_02180_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [4, 5, 6, 7, 23, 24])
def test_lane_counts_by_frames_give_the_same_bits(K):
    import torch
    from paper_1705_02180_amd import scps
    t = np.linspace(0.0, 1.0, K)[:, None]
    path = torch.as_tensor((1 - t) * np.array([[0.0, 5.0]]) + t * np.array([[0.1, 0.2]]), device="cuda")
    xy0 = np.array([[0.0, 5.0]]) + np.random.default_rng(K).normal(0, 1.0, (16390, 2))
    cv0 = np.zeros((16390, 8))
    cv0[:, 1] = cv0[:, 5] = cv0[:, 6] = np.inf

    def run(n):
        xy, cv = torch.as_tensor(xy0[:n].copy(), device="cuda"), torch.as_tensor(cv0[:n].copy(), device="cuda")
        scps.funnel_steps(dict(I.funnel_params(), bias_mode=1), xy, cv, 20, mean_path=path)
        torch.cuda.synchronize()
        return xy.cpu().numpy(), cv.cpu().numpy()

    one = run(16390)
    for n in (4096, 4097, 8192, 8193, 16384):
        got = run(n)
        assert np.array_equal(got[0], one[0][:n]) and np.array_equal(got[1], one[1][:n]), n
