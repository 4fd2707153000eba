"""The split launch with both of its work lists, at sizes that are known to take it:
one step against the FP64 oracle, calls of several lengths against the per-step
path."""
import numpy as np
import pytest

import test_gpu_packed as P
import test_gpu_split as SP
from paper_1705_02180_amd import inputs as I
from test_gpu_large_batches import STEP, one_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1705_02180_amd import scps
    return scps


# the split launch's two work lists: short segments where the long ones are fewer than 48 G
@pytest.mark.parametrize("n,R,contact,G,extra", [
    (200, 4, "all", 8, {}), (200, 64, "all", 4, {}), (971, 128, "all", 2, {}),
    (1600, 64, "all", 4, {"min_seq_sep": 35, "r_cut_contact": 12.0}), (1664, 64, "half", 4, {}),
], ids=["200x4short", "200x64short", "971x128long", "1600x64long", "1664x64long"])
def test_split_step_matches_oracle(S, n, R, contact, G, extra):
    base = dict(I._base_params(), **STEP)
    base.update(extra)
    sy = P._system(n, contact, 23)
    ctx = S.Context.from_workload(I.Workload("g", base, [sy], np.zeros(R, np.int32), 1), params=base)
    assert ctx.get_launch_shape() == ("split", 1, G)
    ctx.close()
    one_step(S, [sy], np.zeros(R, np.int32), base, None, "split", [0, 1, R - 1], 4)


@pytest.mark.parametrize("n,R,contact,over", [
    (971, 128, "all", {}), (1600, 64, "third", {"integrator": 0, "dt": 2e-4}), (200, 4, "all", {})],
    ids=["971x128", "1600x64", "200x4"])
def test_split_calls_follow_the_per_step_path(S, n, R, contact, over):
    """Calls of several lengths with frames, as for the shapes of the split tests."""
    w = SP.workload([n], contact, [0] * R, **over)
    ctx = SP.context(S, w)
    assert ctx.get_launch_shape()[0] == "split"
    ctx.close()
    calls = (1, 2, 0, 3)
    a = SP.run(SP.context(S, w), w, calls, record=2)
    b = SP.run(SP.context(S, w, exec_mode=1), w, calls, record=2)
    disp = np.abs(b[0] - w.initial_x()).max()
    assert np.abs(a[0] - b[0]).max() <= 1e-4 * disp
    if a[1] is not None:
        assert np.abs(a[1] - b[1]).max() <= 1e-4 * np.abs(b[1]).max()
    np.testing.assert_allclose(a[2][:, :2], b[2][:, :2], rtol=1e-5)
    for fa, fb in zip(a[3], b[3]):
        assert np.abs(fa - fb).max() <= 1e-4 * disp
