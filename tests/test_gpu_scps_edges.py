"""GPU parity of the SCPS step at the edges of its kernels' shapes: groups of 1
to 33 replicas (16- and 32-wide matrix work, one to four replicas a pair
wavefront), stacks around every frame count the passes are cut to, and contact
sets of one to a few blocks.  One BAOAB step from rest at kT = 0 gives the
force back as v = c1 dt F / m."""
import math

import numpy as np
import pytest

import oracle as O
from paper_1705_02180_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = 1e-5   # normwise forces, s, and w: the bounds of the parity tests


@pytest.mark.parametrize("R,K,n,nc,seqsep", [
    (1, 2, 70, 70, 0), (7, 16, 66, 64, 0), (8, 17, 130, 65, 0), (9, 31, 90, 90, 35), (15, 32, 64, 64, 0),
    (16, 33, 70, 66, 0), (17, 40, 90, 90, 0), (24, 41, 70, 70, 0), (25, 48, 64, 64, 5), (32, 49, 70, 65, 0),
    (33, 52, 66, 66, 0), (3, 53, 70, 70, 0), (16, 64, 70, 70, 0), (5, 65, 130, 128, 0), (20, 72, 70, 70, 0),
    (16, 73, 70, 70, 0), (2, 80, 66, 66, 35), (31, 81, 66, 66, 0), (12, 96, 66, 66, 0), (18, 97, 66, 66, 0),
    (4, 112, 66, 66, 0), (6, 113, 66, 66, 0), (17, 128, 66, 66, 0)])
def test_scps_step_at_shape_edges(R, K, n, nc, seqsep):
    import torch
    from paper_1705_02180_amd import scps
    p = dict(I._base_params(), integrator=1, kT=0.0, gamma=1e-3, dt=0.002, bias_mode=1, lam=13.5, k_s=50.0, k_w=5.0,
             min_seq_sep=seqsep, seed=1, k_bond=0.0, lj_eps=0.0, dh_prefactor=0.0)   # the bias force alone
    rng = np.random.default_rng(1000 * R + K)
    sy = I.System(n=n, contact_idx=np.sort(rng.choice(n, nc, replace=False)).astype(np.int32),
                  mass=np.full(n, 12.011 * I.AMU, np.float32), charge=rng.normal(0, 0.3, n).astype(np.float32),
                  native=I.compact_native(n, 7), start=I.persistent_start(n, 8))
    ctx = scps.Context(p, [n], [sy.contact_idx], [sy.mass], [sy.charge], np.zeros(R, np.int32))
    ctx.set_reference_map(0, native_xyz=sy.native)
    t = np.linspace(0.0, 1.0, K)[:, None, None, None]
    frames = ((1 - t) * sy.start + t * sy.native + rng.normal(0, 0.5, (K, 2, 3, n))).astype(np.float32)
    stack = ctx.update_reference_from_paths(0, torch.as_tensor(frames.ravel(), device="cuda"), 2, K,
                                            np.ones(2, np.uint8), want_maps=True)
    osys = O.System(n, sy.contact_idx, sy.mass, sy.charge, p, native_xyz=sy.native, stack=stack)
    X = np.stack([frames[(r * (K - 1)) // max(R - 1, 1), r % 2] + rng.normal(0, 0.1, (3, n)) for r in range(R)])
    X = X.astype(np.float32)
    cv0 = np.zeros((R, 8))
    cv0[:, 1] = np.inf
    for r in range(R):
        s, w, *_ = O.tube(X[r].astype(np.float64), sy.contact_idx, stack, osys.Z0, p["lam"], min_sep=seqsep,
                          grads=False)
        cv0[r, 5], cv0[r, 6] = s - 0.05, w - 0.01
    x, cv = torch.as_tensor(X.ravel(), device="cuda"), torch.as_tensor(cv0, device="cuda")
    v = torch.zeros_like(x)
    ctx.step_replicas(x, v, cv, 1)
    ctx.sync()
    V = v.cpu().numpy().reshape(R, 3, n).astype(np.float64) * sy.mass / (math.exp(-p["gamma"] * p["dt"]) * p["dt"])
    CV = cv.cpu().numpy()
    for r in range(R):
        F, _, cvr = O.total_force(p, osys, X[r].astype(np.float64), cv0[r])
        err = np.linalg.norm(V[r] - F, axis=0).max() / np.linalg.norm(F, axis=0).max()
        assert err <= TOL, (r, err)
        assert abs(CV[r, 3] - cvr[3]) <= TOL and abs(CV[r, 4] - cvr[4]) <= TOL * max(1.0, abs(cvr[4])), r
    ctx.close()
