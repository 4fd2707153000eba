"""The packed kernel (chains of 8 and more particles only above 2048 replicas) and
the persistent kernel with 1024 threads (above 128 replicas, or chains of three or
four blocks) in the batch sizes that reach them: forces, z, E_b and T of one step
from rest at kT = 0, noise and short noisy trajectories against the FP64 oracle,
for replicas all over the batch."""
import math

import numpy as np
import pytest

import oracle as O
import test_gpu_packed as P
from paper_1705_02180_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = 1e-5          # normwise forces and z, as in the other parity tests


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1705_02180_amd import scps
    return scps


def one_step(S, systems, rs, base, launch, kernel, sample, base_replicas):
    """One BAOAB step from rest at kT = 0 for a batch that repeats base_replicas
    configurations; the sampled replicas against the oracle, all replicas against the
    first one with their configuration."""
    import torch
    R = len(rs)
    assert all(rs[r] == rs[r % base_replicas] for r in range(R))
    w = I.Workload("step", dict(base), systems, rs, 1)
    X = [P._coil_or_native(systems[rs[r]], r, 90) for r in range(base_replicas)]
    osys = [O.System.from_inputs(sy, base) for sy in systems]
    cvb = np.zeros((base_replicas, 8))
    cvb[:, 1] = np.inf
    for r in range(1, base_replicas):
        o = osys[rs[r]]
        z = O.z_grad(X[r].astype(np.float64), o.cidx, o.native, r_cut=base["r_cut_contact"],
                     min_sep=base["min_seq_sep"], grad=False)
        cvb[r, 1] = 0.7 * z if r % 2 else 1.3 * z
    b = np.arange(R) % base_replicas
    ctx = P._context(S, w, base, launch=launch)
    assert ctx.get_launch_shape()[0] == kernel
    x = P.dev(np.concatenate([X[k].ravel() for k in b]))
    v, cv = torch.zeros_like(x), P.dev(cvb[b], "f64")
    ctx.step_replicas(x, v, cv, 1, step0=3)
    ctx.sync()
    ctx.close()
    V, CV = P.host(v), P.host(cv)
    off = np.concatenate([[0], np.cumsum([3 * systems[s].n for s in rs])])
    c1 = math.exp(-base["gamma"] * base["dt"])
    for r in range(R):
        k = r % base_replicas
        a, f = V[off[r]:off[r + 1]], V[off[k]:off[k + 1]]
        assert np.abs(a - f).max() <= TOL * np.abs(f).max(), r
        assert abs(CV[r, 0] - CV[k, 0]) <= TOL * max(CV[k, 0], 1e-12), r
    for r in sample:
        k, sy, o = r % base_replicas, systems[rs[r]], osys[rs[r]]
        Fg = V[off[r]:off[r + 1]].reshape(3, sy.n).astype(np.float64) * sy.mass.astype(np.float64) / (c1 * base["dt"])
        F, _, cvr = O.total_force(base, o, X[k].astype(np.float64), cvb[k])
        assert P.normwise(Fg, F) <= TOL, (r, P.normwise(Fg, F))
        zs = max(cvr[0], 1e-3 * max(o.Z0, 1e-300))
        assert abs(CV[r, 0] - cvr[0]) <= TOL * zs + 1e-12, r
        assert abs(CV[r, 1] - cvr[1]) <= TOL * max(cvr[1], 1e-3 * max(o.Z0, 1e-300)) + 1e-12, r
        # E_b = k_R (z - z_m)^2 / 2 through its root, a difference of two z-sized numbers
        assert abs(math.sqrt(CV[r, 2]) - math.sqrt(cvr[2])) <= 2 * TOL * zs * math.sqrt(0.5 * base["k_R"]) + 1e-12, r
        # sqrt(T) is a weighted norm of the bias force
        _, _, cvs, _ = O.steps(base, o, r, X[k].astype(np.float64), np.zeros(X[k].shape), cvb[k], 1, step0=3)
        tol_t = TOL * np.linalg.norm(F, axis=0).max() * math.sqrt(
            base["dt"] * np.sum(1.0 / (sy.mass.astype(np.float64) * base["gamma"])))
        assert abs(math.sqrt(CV[r, 7]) - math.sqrt(cvs[7])) <= tol_t, r


STEP = dict(integrator=1, kT=0.0, gamma=1e-3, dt=0.002, k_R=2e-2)


@pytest.mark.parametrize("waves", [1, 2, 8])
@pytest.mark.parametrize("name,sizes,contact,_,pattern,extra", [c for c in P.CASES if max(c[1]) >= 8],
                         ids=[c[0] for c in P.CASES if max(c[1]) >= 8])
def test_packed_step_in_a_large_batch_matches_oracle(S, name, sizes, contact, _, pattern, extra, waves):
    """2053 and more replicas (a ragged last wavefront and workgroup) on the packed kernel."""
    base = dict(I._base_params(), **STEP)
    base.update(extra)
    pattern = pattern or [0] * 12
    R = 2053 + len(pattern) - 2053 % len(pattern) + 1
    rs = np.asarray(pattern, np.int32)[np.arange(R) % len(pattern)]
    systems = [P._system(n, contact, 40 + 7 * i) for i, n in enumerate(sizes)]
    one_step(S, systems, rs, base, (2, waves), "packed", list(range(len(pattern))) + [1000, 1001, R - 2, R - 1],
             len(pattern))


@pytest.mark.parametrize("n,R,contact,extra", [
    (560, 130, "half", {}), (560, 129, "all", {"min_seq_sep": 35, "r_cut_contact": 12.0, "r_cut_nb": 10.0}),
    (130, 200, "all", {}), (192, 3, "tail", {"min_seq_sep": 5}), (320, 140, "half", {"lj_eps": 0.0}),
    (700, 131, "tail", {"dh_prefactor": 0.0}),
], ids=["560x130", "560x129cut", "130x200", "192x3", "320x140", "700x131"])
def test_persistent_1024_step_matches_oracle(S, n, R, contact, extra):
    base = dict(I._base_params(), **STEP)
    base.update(extra)
    k = min(R, 4)
    one_step(S, [P._system(n, contact, 17)], np.zeros(R, np.int32), base, None, "persistent",
             sorted({0, 1, k - 1, R // 2, R - 1}), k)


@pytest.mark.parametrize("waves", [1, 4, 8])
@pytest.mark.parametrize("integrator", [0, 1], ids=["overdamped", "baoab"])
@pytest.mark.parametrize("sizes", [[20], [13, 20], [64, 33]], ids=str)
def test_packed_noisy_trajectories_match_oracle(S, sizes, integrator, waves):
    """Five steps with noise on the packed kernel, replicas at both ends and in the
    middle of a batch of 2053: positions, z, E_b and T."""
    base = dict(I._base_params(), integrator=integrator, k_R=2e-2)
    if integrator == 0:
        base.update(dt=2e-4)
    R, steps = 2053, 5
    rs = np.arange(R, dtype=np.int32) % len(sizes)
    systems = [P._system(n, "half", 40 + 7 * i) for i, n in enumerate(sizes)]
    w = I.Workload("traj", dict(base), systems, rs, 1)
    ctx = P._context(S, w, base, launch=(2, waves))
    assert ctx.get_launch_shape()[0] == "packed"
    x0, v0, cv0 = w.initial_x(), w.initial_v(3), w.initial_cvstate()
    x, cv = P.dev(x0), P.dev(cv0, "f64")
    v = P.dev(v0) if integrator else None
    ctx.step_replicas(x, v, cv, steps, step0=17)
    ctx.sync()
    ctx.close()
    got, CV = P.host(x), P.host(cv)
    off = np.concatenate([[0], np.cumsum([3 * systems[s].n for s in rs])])
    for r in (0, 1, 2, 3, 1022, 1023, R - 2, R - 1):
        sy = systems[rs[r]]
        a, b = off[r], off[r + 1]
        o = O.System.from_inputs(sy, base)
        X = x0[a:b].reshape(3, sy.n).astype(np.float64)
        V = v0[a:b].reshape(3, sy.n).astype(np.float64) if integrator else np.zeros((3, sy.n))
        xo, _, cvo, _ = O.steps(base, o, r, X, V, cv0[r], steps, step0=17)
        disp = np.abs(xo - X).max()
        assert np.abs(got[a:b].reshape(3, sy.n) - xo).max() <= 1e-4 * disp, r
        np.testing.assert_allclose(CV[r, :2], cvo[:2], rtol=1e-5)
        zs = 1e-4 * cvo[0]
        assert abs(math.sqrt(CV[r, 2]) - math.sqrt(cvo[2])) <= zs * math.sqrt(0.5 * base["k_R"]), r
        assert abs(math.sqrt(CV[r, 7]) - math.sqrt(cvo[7])) <= 1e-3 * math.sqrt(cvo[7]) + zs, r


@pytest.mark.parametrize("waves", [1, 8])
def test_packed_noise_in_a_large_batch_matches_oracle_philox(S, waves):
    """Free overdamped particles with unit noise amplitude, a 64-bit step."""
    import torch
    n, R = 30, 2060
    p = dict(I._base_params(), integrator=0, dt=1.0, gamma=1.0, kT=0.5, k_bond=0.0, lj_eps=0.0,
             dh_prefactor=0.0, k_R=0.0, seed=0x1234_5678_9ABC)
    sy = P._system(n, "half", 3)
    sy.mass[:] = 1.0
    w = I.Workload("noise", dict(p), [sy], np.zeros(R, dtype=np.int32), 1)
    ctx = S.Context.from_workload(w, params=p, replica_base=7)
    ctx.set_reference_map(0, native_xyz=sy.native)
    ctx.set_launch(2, waves)
    assert ctx.get_launch_shape()[0] == "packed"
    x = torch.zeros(3 * n * R, dtype=torch.float32, device="cuda")
    cv = P.dev(np.tile([0, np.inf, 0, 0, 0, np.inf, np.inf, 0], (R, 1)), "f64")
    step = (1 << 32) + 5
    ctx.step_replicas(x, None, cv, 1, step0=step)
    got = P.host(x).reshape(R, 3, n)
    ctx.close()
    for r in (0, 1, 2, 15, 1024, R - 2, R - 1):
        want = O.normals(p["seed"], np.arange(n), 7 + r, step).T
        np.testing.assert_allclose(got[r], want, rtol=1e-6, atol=1e-6)
