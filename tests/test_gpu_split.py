"""The split rMD launch (several workgroups per replica, one launch per step)
against the per-step path, and its bookkeeping over calls."""
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


def dev(a, dtype="f32"):
    import torch
    t = {"f32": torch.float32, "f64": torch.float64}[dtype]
    return torch.as_tensor(np.ascontiguousarray(a), dtype=t, device="cuda")


def host(t):
    return t.detach().cpu().numpy()


def workload(sizes, contact, rsys, **over):
    rng = np.random.default_rng(sum(sizes))
    systems = []
    for n in sizes:
        idx = {"all": np.arange(n), "third": np.arange(0, n, 3), "none": np.arange(0)}[contact]
        systems.append(I.System(n=n, contact_idx=idx.astype(np.int32), mass=np.full(n, 12.011 * I.AMU, np.float32),
                                charge=rng.normal(0, 0.3, n).astype(np.float32), native=I.compact_native(n, 7),
                                start=I.persistent_start(n, 8)))
    return I.Workload("split", dict(I._base_params(), **over), systems, np.asarray(rsys, np.int32), 1)


def context(S, w, exec_mode=0):
    ctx = S.Context.from_workload(w, params=w.params, exec_mode=exec_mode)
    for s, sy in enumerate(w.systems):
        ctx.set_reference_map(s, native_xyz=sy.native)
    return ctx


def run(ctx, w, calls, record=0):
    """States after the calls, and the frames recorded in them."""
    import torch
    x, v, cv = dev(w.initial_x()), dev(w.initial_v(3)), dev(w.initial_cvstate(), "f64")
    v = v if w.params["integrator"] == 1 else None
    step, frames = 5, []
    for m in calls:
        fr = torch.zeros((m // record + 1, x.numel()), device="cuda") if record else None
        ctx.step_replicas(x, v, cv, m, step0=step, record_every=record, frames=fr)
        step += m
        frames.append(host(fr) if record else None)
    ctx.sync()
    return host(x), None if v is None else host(v), host(cv), frames


CASES = [
    # sizes, contact set, replicas' systems, parameters
    ([161], "all", [0] * 4, {}),                                     # the fewest blocks, 256 / R clipped by the items
    ([384], "third", [0] * 3, {"integrator": 0, "dt": 2e-4}),       # whole blocks, overdamped, no velocities
    ([560], "all", [0] * 128, {}),                                   # two workgroups per replica
    ([560, 200], "third", [0, 1, 1, 0, 1], {}),                      # a chain with fewer items than workgroups
    ([700], "none", [0] * 2, {"dh_prefactor": 0.0}),                # no contact pairs: z = 0
    ([450], "all", [0] * 2, {"lj_eps": 0.0, "r_cut_contact": 12.0, "min_seq_sep": 35}),
    ([1664], "third", [0] * 2, {}),                                  # the longest chain of the 1024-thread launch
]


@pytest.mark.parametrize("sizes,contact,rsys,over", CASES, ids=["161x4", "384x3", "560x128", "560+200", "700none",
                                                                  "450cut", "1664x2"])
def test_split_equals_the_per_step_path(S, sizes, contact, rsys, over):
    """Calls of 1, 2, 3 and 0 steps leave the three accumulators at every phase."""
    w = workload(sizes, contact, rsys, **over)
    calls = (1, 2, 3, 0, 1, 4)
    a = run(context(S, w), w, calls, record=2)
    b = run(context(S, w, exec_mode=1), w, calls, record=2)
    x0 = w.initial_x()
    disp = np.abs(b[0] - x0).max()
    assert np.abs(a[0] - b[0]).max() <= 1e-4 * disp
    if a[1] is not None:
        assert np.abs(a[1] - b[1]).max() <= 1e-4 * np.abs(b[1]).max()
    np.testing.assert_allclose(a[2][:, :2], b[2][:, :2], rtol=1e-5)
    # E_b = k_R (z - z_m)^2 / 2 and T ~ (z - z_m)^2: compare roots, differences of z-sized numbers
    for k, s in ((2, np.sqrt(0.5 * w.params["k_R"])), (7, None)):
        ra, rb = np.sqrt(a[2][:, k]), np.sqrt(b[2][:, k])
        assert np.abs(ra - rb).max() <= (1e-4 * s * b[2][:, 0].max() if s else 1e-3 * rb.max() + 1e-12)
    for fa, fb in zip(a[3], b[3]):
        assert np.abs(fa - fb).max() <= 1e-4 * disp


def test_split_call_replays_from_a_captured_graph(S):
    """A captured call holds kernels alone and leaves its buffers as it found
    them: replays continue the trajectory that the launches give (kT = 0)."""
    import torch
    w = workload([560], "third", [0] * 4, kT=0.0)
    ctx = context(S, w)
    x, v, cv = dev(w.initial_x()), dev(w.initial_v(3)), dev(w.initial_cvstate(), "f64")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ctx.step_replicas(x, v, cv, 2)
    torch.cuda.synchronize()
    x.copy_(dev(w.initial_x())), v.copy_(dev(w.initial_v(3))), cv.copy_(dev(w.initial_cvstate(), "f64"))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        ctx.step_replicas(x, v, cv, 2)
    other = torch.zeros(1000, device="cuda")
    for k in range(4):
        g.replay()
        other += 1
        torch.cuda.synchronize()
        ref = context(S, w)
        xr, vr, cvr = dev(w.initial_x()), dev(w.initial_v(3)), dev(w.initial_cvstate(), "f64")
        ref.step_replicas(xr, vr, cvr, 2 * (k + 1))
        ref.sync()
        disp = np.abs(host(xr) - w.initial_x()).max()
        assert np.abs(host(x) - host(xr)).max() <= 1e-4 * disp, k
        np.testing.assert_allclose(host(cv)[:, :2], host(cvr)[:, :2], rtol=1e-5)
        ref.close()
    ctx.close()


def test_split_reports_a_nonfinite_replica(S):
    w = workload([400], "all", [0] * 3)
    ctx = context(S, w)
    X = w.initial_x()
    X[3 * 400 + 17] = np.nan
    ctx.step_replicas(dev(X), dev(w.initial_v(3)), dev(w.initial_cvstate(), "f64"), 2)
    with pytest.raises(S.ScpsError) as e:
        ctx.sync()
    assert e.value.status == -6 and "[1]" in str(e.value)
