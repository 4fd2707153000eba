"""Short chains in small batches (one wavefront per replica) against the per-step
path, and the packed kernel, which larger batches take, against the small ones."""
import numpy as np
import pytest

from paper_1705_02180_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1705_02180_amd import scps
    return scps


def systems(sizes):
    out = []
    for n in sizes:
        rng = np.random.default_rng(n)
        out.append(I.System(n=n, contact_idx=np.sort(rng.choice(n, max(2, n - n // 4), replace=False)).astype(np.int32),
                            mass=rng.uniform(0.1, 0.2, n).astype(np.float32),
                            charge=rng.normal(0, 0.3, n).astype(np.float32), native=I.compact_native(n, 7),
                            start=I.persistent_start(n, 8)))
    return out


def run(S, sizes, rsys, steps, exec_mode=0, **over):
    """x, v, cv after the steps, and the frames of every second one."""
    import torch
    p = dict(I._base_params(), **over)
    w = I.Workload("wide", p, systems(sizes), np.asarray(rsys, np.int32), 1)
    ctx = S.Context.from_workload(w, params=p, exec_mode=exec_mode)
    for s, sy in enumerate(w.systems):
        ctx.set_reference_map(s, native_xyz=sy.native)
    x = torch.as_tensor(w.initial_x(), device="cuda")
    v = torch.as_tensor(w.initial_v(3), device="cuda") if p["integrator"] == 1 else None
    cv = torch.as_tensor(w.initial_cvstate(), device="cuda")
    fr = torch.zeros((steps // 2 + 1, x.numel()), device="cuda")
    ctx.step_replicas(x, v, cv, steps, step0=7, record_every=2, frames=fr)
    ctx.sync()
    ctx.close()
    return [None if t is None else t.cpu().numpy() for t in (x, v, cv, fr)] + [w.initial_x()]


@pytest.mark.parametrize("integrator", [0, 1])
@pytest.mark.parametrize("sizes", [[8], [9], [10], [13], [16], [21], [22], [31], [32], [33], [47], [48], [20, 11, 48]],
                         ids=str)
def test_wide_equals_the_per_step_path(S, sizes, integrator):
    over = dict(integrator=integrator, min_seq_sep=3, nb_excl=2)
    if integrator == 0:
        over.update(dt=2e-4)
    rsys = np.arange(5) % len(sizes)
    a, b = run(S, sizes, rsys, 9, **over), run(S, sizes, rsys, 9, exec_mode=1, **over)
    disp = np.abs(b[0] - b[4]).max()
    assert np.abs(a[0] - b[0]).max() <= 1e-4 * disp
    assert np.abs(a[3] - b[3]).max() <= 1e-4 * disp
    if integrator:
        assert np.abs(a[1] - b[1]).max() <= 1e-4 * np.abs(b[1]).max()
    np.testing.assert_allclose(a[2][:, :2], b[2][:, :2], rtol=1e-5, atol=1e-12)


@pytest.mark.parametrize("sizes", [[2], [5], [7], [8], [20], [32], [31, 6], [33], [48]], ids=str)
def test_packed_batch_equals_a_small_one(S, sizes):
    """2049 replicas run packed; their first ones agree with a batch of 4."""
    n = len(sizes)
    a, b = run(S, sizes, np.arange(2049) % n, 9), run(S, sizes, np.arange(4) % n, 9)
    m = b[0].size
    disp = np.abs(b[0] - b[4]).max()
    assert np.abs(a[0][:m] - b[0]).max() <= 1e-4 * disp
    assert np.abs(a[3][:, :m] - b[3]).max() <= 1e-4 * disp
    assert np.abs(a[1][:m] - b[1]).max() <= 1e-4 * np.abs(b[1]).max()
    np.testing.assert_allclose(a[2][:4, :2], b[2][:, :2], rtol=1e-5, atol=1e-12)
