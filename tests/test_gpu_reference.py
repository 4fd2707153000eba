"""GPU parity of the reference-map update: the path means at every remainder of
the path groups, with coordinates far outside a chain's range, and the frame
distances of the stack at the edges of its blocks of frames."""
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


def chain(S, n, contact_idx, R, **over):
    p = dict(I._base_params(), lam=13.5, **over)
    rng = np.random.default_rng(n)
    sy = I.System(n=n, contact_idx=np.asarray(contact_idx, np.int32), mass=np.full(n, 12.011 * I.AMU, np.float32),
                  charge=np.zeros(n, np.float32), native=I.compact_native(n, 3), start=I.persistent_start(n, 4))
    ctx = S.Context(p, [n], [sy.contact_idx], [sy.mass], [sy.charge], np.zeros(R, np.int32))
    ctx.set_reference_map(0, native_xyz=sy.native)
    return ctx, sy, p, rng


def paths(sy, K, n_paths, rng):
    t = np.linspace(0.0, 1.0, K)[:, None, None, None]
    f = (1 - t) * sy.start + t * sy.native
    return (f + rng.normal(0, 0.8, (K, n_paths, 3, sy.n))).astype(np.float32)


@pytest.mark.parametrize("cut", [0.0, 12.0])
@pytest.mark.parametrize("far", [None, 1.0e10, 1.0e18])
@pytest.mark.parametrize("n_succ", [1, 2, 3, 4, 7, 8, 13])
def test_path_mean_at_every_group_size(S, n_succ, far, cut):
    """Path groups of 4, 2 and 1 and batches of 8; far: one path's particles lie
    that far apart, where four denominators together would overflow at 1e18."""
    import torch
    n, K = 70, 3
    ctx, sy, p, rng = chain(S, n, np.arange(1, 70), 1, r_cut_contact=cut)
    fr = paths(sy, K, n_succ + 2, rng)
    if far:
        fr[1, n_succ // 2] = (rng.normal(0, 1, (3, n)) * far).astype(np.float32)
    succ = np.ones(n_succ + 2, np.uint8)
    succ[[0, n_succ + 1]] = 0
    if n_succ == 1:
        fr[:, 1] = fr[:, n_succ // 2]
    maps = ctx.update_reference_from_paths(0, torch.as_tensor(fr.ravel(), device="cuda"), n_succ + 2, K, succ,
                                           want_maps=True)
    x = fr[:, 1:n_succ + 1].astype(np.float64)[..., sy.contact_idx]
    a, b = np.triu_indices(len(sy.contact_idx), 1)
    r2 = ((x[..., a] - x[..., b]) ** 2).sum(2)
    q = r2 / 7.5 ** 2
    C = (1 + q + q * q) / (1 + q + q * q + q ** 3 + q ** 4)
    want = np.where((cut > 0) & (r2 > cut * cut), 0.0, C).mean(1)
    np.testing.assert_allclose(maps, want, rtol=1e-12, atol=1e-15)
    ctx.close()


@pytest.mark.parametrize("K,nc", [(2, 64), (6, 65), (7, 3), (64, 66), (65, 66), (72, 130), (128, 66)])
def test_tube_of_new_stack_at_block_edges(S, K, nc):
    """s and w carry the pair-major stack and every G_jk: K at the edges of the
    blocks of 6 frames, of the batches (64) and the largest stack."""
    import torch
    n, R = 140, 5
    ctx, sy, p, rng = chain(S, n, np.sort(np.random.default_rng(K).choice(n, nc, replace=False)), R)
    fr = paths(sy, K, 2, rng)
    stack = ctx.update_reference_from_paths(0, torch.as_tensor(fr.ravel(), device="cuda"), 2, K,
                                            np.ones(2, np.uint8), want_maps=True)
    X = np.stack([fr[(r * (K - 1)) // (R - 1), r % 2] + rng.normal(0, 0.3, (3, n)) for r in range(R)])
    X = X.astype(np.float32)
    s = torch.zeros(R, dtype=torch.float64, device="cuda")
    w = torch.zeros_like(s)
    ctx.eval_tube(0, torch.as_tensor(X.ravel(), device="cuda"), s, w)
    ctx.sync()
    Z0 = O.System.from_inputs(sy, p).Z0
    for r in range(R):
        so, wo, *_ = O.tube(X[r].astype(np.float64), sy.contact_idx, stack, Z0, 13.5, grads=False)
        assert abs(s[r].item() - so) <= 1e-5 and abs(w[r].item() - wo) <= 1e-5 * max(1.0, abs(wo))
    ctx.close()
