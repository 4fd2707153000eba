"""The distance pass's sums in one set and in 16 (where many workgroups meet on a
group of replicas): the same results, and no more device memory than the batch
needs."""
import numpy as np
import pytest

import oracle as O
from paper_1705_02180_amd import inputs as I

pytestmark = pytest.mark.gpu
K = 5


def chain(N):
    rng = np.random.default_rng(3)
    sy = I.System(n=N, contact_idx=np.arange(N, dtype=np.int32), mass=np.full(N, 0.12, np.float32),
                  charge=rng.normal(0, 0.3, N).astype(np.float32), native=I.compact_native(N, 7),
                  start=I.persistent_start(N, 8))
    t = np.linspace(0.0, 1.0, K)[:, None, None, None]
    frames = ((1 - t) * sy.start + t * sy.native + rng.normal(0, 0.4, (K, 2, 3, N))).astype(np.float32)
    return sy, frames


def context(R, bias_mode, N=150):
    import torch
    from paper_1705_02180_amd import scps
    sy, frames = chain(N)
    # frames between the start and the native fold overlap: no Lennard-Jones or charges
    p = dict(I._base_params(), bias_mode=bias_mode, lam=13.5, k_s=50.0, k_w=5.0, lj_eps=0.0, dh_prefactor=0.0)
    ctx = scps.Context(p, [N], [sy.contact_idx], [sy.mass], [sy.charge], np.zeros(R, np.int32))
    ctx.set_reference_map(0, native_xyz=sy.native)
    maps = ctx.update_reference_from_paths(0, torch.as_tensor(frames.ravel(), device="cuda"), 2, K,
                                           np.ones(2, np.uint8), want_maps=True)
    rng = np.random.default_rng(11)
    X = np.stack([frames[r % K, r % 2] + rng.normal(0, 0.1, (3, N)) for r in range(R)]).astype(np.float32)
    return ctx, sy, p, maps, X


# 150 particles are 6 tiles a group: a batch of 4 takes them with 96 workgroups (16 sets); 66, 102 and 198
# tiles take 8, 4 and 2 workgroups each (16 sets, 1 and 1)
@pytest.mark.parametrize("R", [352, 520, 1050])
def test_one_set_and_many_give_the_same_tube_variables(R):
    import torch
    out = []
    for reps in (4, R):
        ctx, sy, p, maps, X = context(reps, 0)
        x = torch.as_tensor(X.ravel(), device="cuda")
        s, w = (torch.empty(reps, dtype=torch.float64, device="cuda") for _ in range(2))
        for _ in range(2):                       # the second pass starts from sums that the first one cleared
            s.zero_(), w.zero_()
            ctx.eval_tube(0, x, s, w)
            ctx.sync()
            out.append((s.cpu().numpy(), w.cpu().numpy()))
        ctx.close()
    osys = O.System(sy.n, sy.contact_idx, sy.mass, sy.charge, p, native_xyz=sy.native, stack=maps)
    for r in (0, 1, 31, 32, R - 1):
        so, wo, *_ = O.tube(X[r].astype(np.float64), sy.contact_idx, maps, osys.Z0, p["lam"], grads=False)
        assert abs(out[2][0][r] - so) <= 1e-5 and abs(out[2][1][r] - wo) <= 1e-5, r
    # another order of at most 11175 float64 terms: 2e-12 of a distance, 13.5 times that in an exponent
    for s, w in out[1:]:
        np.testing.assert_allclose(s[:4], out[0][0], rtol=0, atol=1e-9)
        np.testing.assert_allclose(w[:4], out[0][1], rtol=0, atol=1e-9)


def test_one_set_and_many_step_alike():
    import torch
    R, N = 520, 150
    out = []
    for reps in (4, R):
        ctx, sy, p, maps, X = context(reps, 1)
        cv0 = np.zeros((reps, 8))
        cv0[:, 1], cv0[:, 5], cv0[:, 6] = np.inf, -0.2, -1.0
        x, cv = torch.as_tensor(X.ravel(), device="cuda"), torch.as_tensor(cv0, device="cuda")
        v = torch.zeros_like(x)
        ctx.step_replicas(x, v, cv, 6, step0=3)
        ctx.sync()
        ctx.close()
        out.append((x.cpu().numpy()[:12 * N], v.cpu().numpy()[:12 * N], cv.cpu().numpy()[:4]))
    a, b = out
    disp = np.abs(a[0] - X[:4].ravel()).max()
    assert np.abs(a[0] - b[0]).max() <= 1e-4 * disp
    assert np.abs(a[1] - b[1]).max() <= 1e-4 * np.abs(a[1]).max()
    np.testing.assert_allclose(a[2][:, 3:5], b[2][:, 3:5], rtol=1e-5, atol=1e-7)


def test_tube_evaluation_of_many_short_chains_takes_one_set():
    """16384 chains of one tile: 17 MB of sums (16 sets would be 268 MB)."""
    import torch

    def grown(R):
        ctx, _, _, _, X = context(R, 0, N=20)
        x = torch.as_tensor(X.ravel(), device="cuda")
        s = torch.empty(R, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        ctx.eval_tube(0, x, s)
        ctx.sync()
        used = before - torch.cuda.mem_get_info()[0]
        ctx.close()
        return used

    grown(8192)                                   # the kernels are loaded
    assert grown(16384) <= 64 << 20
