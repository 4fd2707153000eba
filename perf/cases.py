"""Performance cases of the batched rMD / SCPS stepping library.

Each case is one call sequence that a program built on the library makes on
the GPU, through the package's public entry points, at the sizes of the
repository's own workloads (the 20-bead, 560-, 3000- and 6000-particle
chains, the uneven batch, the funnel of the toy model) and between them.

``prepare`` makes what the program holds beforehand (coordinates, velocities,
the context with its reference maps), ``run`` is one call, ``work`` the bytes
and operations the call cannot do without, and ``exact`` the same results in
plain float64 torch.

Collective variables are sums of float32 pair terms kept in float64 slots; the
programs record them in float32, beside the float32 coordinates and frames.
"""
import math

import numpy as np
import torch

from paper_1705_02180_amd import scps

LATTICE = 3.8
AMU = 0.01
KB = 0.0083144626
BASE = dict(integrator=1, bias_mode=0, dt=0.002, gamma=1.0, kT=KB * 300.0, k_bond=100.0, r_bond=LATTICE,
            lj_eps=1.0, lj_sigma=4.0, dh_prefactor=1389.35458 / 80.0, dh_kappa=0.1, nb_excl=2, min_seq_sep=0,
            r0_contact=7.5, r_cut_contact=0.0, r_cut_nb=0.0, k_R=1e-4, lam=13.5, k_s=2.5, k_w=2.5e-4, seed=0)
FUNNEL = dict(A1=30.0, A2=20.0, A3=6.0, s1=1.0, s2=2.0, s3=0.5, w=0.03, xm=1.5, ym=0.0, kT=0.3, mob_dt=0.02,
              k_R=70.0, lam=0.3, k_s=3.0, k_w=3.0)
INF = float("inf")


def device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest ensemble anybody steps: 16 short overdamped chains, a block of steps per call
        # (latency: 16 replicas cannot fill the chip)
        dict(name="rmd 16x20", kind="rmd", n=20, replicas=16, steps=100, reduced=1, heavy=0, cut=0.0),
        # the same chain as a large ensemble (throughput of the packed kernel)
        dict(name="rmd 16384x20", kind="rmd", n=20, replicas=16384, steps=100, reduced=1, heavy=0, cut=0.0),
        # one initial condition of the protocol: 20 trial paths of a Fip35-sized chain (560 particles,
        # 280 in the contact set)
        dict(name="rmd 20x560", kind="rmd", n=560, replicas=20, steps=20, reduced=0, heavy=1, cut=0.0),
        # the same chain as a batch that fills the chip
        dict(name="rmd 256x560", kind="rmd", n=560, replicas=256, steps=20, reduced=0, heavy=1, cut=0.0),
        # chains of odd lengths, each with its own native map, on the per-step path
        dict(name="rmd uneven 128", kind="uneven", chains=128, n_min=200, n_max=3000, steps=4),
        # the serpin-sized chain with both cutoffs: neighbour lists and their rebuilds
        dict(name="rmd 32x6000 cutoff", kind="rmd", n=6000, replicas=32, steps=20, reduced=0, heavy=0, cut=12.0),
        # differentiable z and E_b, forward and backward, one native map per chain
        dict(name="zbias 64x3000", kind="zbias", n=3000, chains=64, grad=1),
        # an SCPS iteration's steps on the Fip35-sized chain, 51 frames (one every 200 of 10^4 steps)
        dict(name="scps 32x560 51f", kind="scps", n=560, replicas=32, frames=51, steps=10, heavy=1),
        # the stack of a full protocol path (about 72 frames) on a middle-sized chain
        dict(name="scps 20x1501 72f", kind="scps", n=1501, replicas=20, frames=72, steps=4, heavy=0),
        # the headline: SCPS steps of 32 serpin-sized chains against 51 frames
        dict(name="scps 32x6000 51f", kind="scps", n=6000, replicas=32, frames=51, steps=2, heavy=0),
        # between two iterations: the mean maps of the successful paths, then s and w of the replicas
        dict(name="mean map 32x6000 51f", kind="mean", n=6000, replicas=32, frames=51, heavy=0, maps=0),
        # the toy model's tube iteration, 51 mean-path frames
        dict(name="funnel 262144 51f", kind="funnel", n=262144, frames=51, steps=50, tube=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["packed", "rmd", "cutoff", "uneven", "zbias", "z", "scps", "mean", "funnel"])
    if kind == "packed":
        return dict(kind="rmd", n=rng.randint(2, 64), replicas=_log(rng, 16, 16384), steps=rng.randint(10, 100),
                    reduced=rng.randint(0, 1), heavy=0, cut=0.0)
    if kind == "rmd":
        n = _log(rng, 65, 3000)
        top = max(16, min(512, int(256 * (560 / n) ** 2)))
        return dict(kind="rmd", n=n, replicas=_log(rng, 8, top), steps=rng.randint(4, 20), reduced=0,
                    heavy=rng.randint(0, 1), cut=0.0)
    if kind == "cutoff":
        n = _log(rng, 560, 6000)
        return dict(kind="rmd", n=n, replicas=rng.randint(8, 32), steps=rng.randint(10, 20), reduced=0,
                    heavy=rng.randint(0, 1), cut=round(rng.uniform(9.0, 12.0), 2))
    if kind == "uneven":
        lo = _log(rng, 100, 600)
        return dict(kind="uneven", chains=rng.randint(16, 96), n_min=lo, n_max=rng.randint(lo + 100, 3000),
                    steps=rng.randint(2, 4))
    if kind in ("zbias", "z"):
        n = _log(rng, 128, 3000)
        return dict(kind="zbias", n=n, chains=_log(rng, 4, 64), grad=int(kind == "zbias"))
    if kind == "scps":
        n = _log(rng, 150, 6000)
        return dict(kind="scps", n=n, replicas=rng.randint(4, 32), frames=rng.randint(9, 51 if n > 3000 else 72),
                    steps=1 if n > 3000 else rng.randint(2, 8), heavy=rng.randint(0, 1))
    if kind == "mean":
        n = _log(rng, 150, 4000)         # small chains also take the maps back to the host
        return dict(kind="mean", n=n, replicas=rng.randint(4, 32), frames=rng.randint(9, 72), heavy=rng.randint(0, 1),
                    maps=int(n <= 560))
    return dict(kind="funnel", n=_log(rng, 1000, 262144), frames=rng.randint(9, 72), steps=rng.randint(20, 50),
                tube=rng.randint(0, 1))


# ---------------------------------------------------------------------------
# inputs (drawn, no method arithmetic)
# ---------------------------------------------------------------------------
def _compact(n):
    """A compact lattice walk: a snake through an L x L x Lz box, [3][n]."""
    L = max(2, int(math.ceil(n ** (1.0 / 3.0))))
    g = np.arange(n)
    z, rest = g // (L * L), g % (L * L)
    rest = np.where(z % 2 == 1, L * L - 1 - rest, rest)
    y, x = rest // L, rest % L
    x = np.where(y % 2 == 1, L - 1 - x, x)
    xyz = np.stack([x, y, z]).astype(np.float64) * LATTICE
    return xyz - xyz.mean(axis=1, keepdims=True)


def _extended(n, run):
    """A flat serpentine of straight runs two lattice spacings apart, [3][n]."""
    per = run + 2                        # run beads in x, then two connecting bonds in y
    g = np.arange(n)
    row, k = g // per, g % per
    x = np.minimum(k, run - 1)
    x = np.where(row % 2 == 1, run - 1 - x, x)
    y = 3 * row + np.maximum(k - (run - 1), 0)
    xyz = np.stack([x, y, np.zeros(n, dtype=np.int64)]).astype(np.float64) * LATTICE
    return xyz - xyz.mean(axis=1, keepdims=True)


def _chain(n, heavy, reduced, rng):
    """(contact_idx, mass, charge) of one chain."""
    if heavy:
        on = np.arange(n) % 16 < 8
        return (np.nonzero(on)[0].astype(np.int32), (np.where(on, 12.011, 1.008) * AMU).astype(np.float32),
                rng.normal(0.0, 0.3, n).astype(np.float32))
    mass = np.ones(n, np.float32) if reduced else np.full(n, 12.011 * AMU, np.float32)
    charge = np.zeros(n, np.float32) if reduced else rng.normal(0.0, 0.3, n).astype(np.float32)
    return np.arange(n, dtype=np.int32), mass, charge


def _sizes(case):
    """Chain lengths of a batch: the case's own, whatever the inputs."""
    if case["kind"] == "zbias":
        return np.full(case["chains"], case["n"])
    rng = np.random.default_rng([case["chains"], case["n_min"], case["n_max"]])
    return rng.integers(case["n_min"], case["n_max"] + 1, case["chains"])


def _inputs(case, seed):
    """What a case's inputs are made of, from the seed alone (host arrays)."""
    rng = np.random.default_rng([int(seed), 20170502])
    kind = case["kind"]
    d = dict(seed=int(seed) + 1)
    if kind == "funnel":
        n, K = case["n"], case["frames"]
        t = np.linspace(0.0, 1.0, K)[:, None]
        d["path"] = (1 - t) * np.array([[0.0, 5.0]]) + t * np.array([[0.1, 0.2]]) + rng.normal(0, 0.05, (K, 2))
        u = rng.random((n, 1))           # trajectories under way along the path
        d["xy"] = (1 - u) * np.array([[0.0, 5.0]]) + u * np.array([[0.1, 0.2]]) + rng.normal(0, 0.3, (n, 2))
        return d
    if kind in ("uneven", "zbias"):
        R = case["chains"]
        sizes = _sizes(case)
        d["chains"] = [_chain(int(n), 0, 0, rng) for n in sizes]
        d["native"] = [_compact(int(n)) + rng.normal(0, 0.2, (3, int(n))) for n in sizes]
        d["x"] = [(_extended(int(n), int(rng.integers(8, 40))) + rng.normal(0, 0.05, (3, int(n)))).astype(np.float32)
                  for n in sizes]
        d["v"] = [(rng.normal(size=(3, len(m))) * np.sqrt(BASE["kT"] / m)).astype(np.float32)
                  for _, m, _ in d["chains"]]
        return d
    n, R = case["n"], case["replicas"]
    d["chains"] = [_chain(n, case["heavy"], case.get("reduced", 0), rng)]
    mass = d["chains"][0][1]
    native = _compact(n) + rng.normal(0, 0.05, (3, n))
    d["native"] = [native]
    if kind == "rmd":
        base = native if case["cut"] > 0 else _extended(n, 24)
        d["x"] = (base[None] + rng.normal(0, 0.05, (R, 3, n))).astype(np.float32)
    else:
        # replicas near the folded end of the paths
        scale = rng.uniform(1.0, 1.15, (R, 1, 1))
        d["x"] = (native[None] * scale + rng.normal(0, 0.1, (R, 3, n))).astype(np.float32)
    d["v"] = (rng.normal(size=(R, 3, n)) * np.sqrt(BASE["kT"] / mass)).astype(np.float32)
    if kind in ("scps", "mean"):
        # recorded paths from an expanded to the folded state; the steps' stack averages 4 of them
        K, paths = case["frames"], (R if kind == "mean" else 4)
        t = np.linspace(0.0, 1.0, K)[:, None, None, None]
        f = native[None, None] * (1.0 + 0.6 * (1.0 - t)) * rng.uniform(0.97, 1.03, (1, paths, 1, 1))
        d["frames"] = f.astype(np.float32)
        d["frames"] += rng.standard_normal((K, paths, 3, n), dtype=np.float32) * np.float32(0.3)
        d["success"] = np.ones(paths, np.uint8)
        if kind == "mean":
            d["success"][rng.integers(0, paths, max(1, paths // 8))] = 0   # some paths did not reach the native state
            d["success"][0] = 1
    return d


def _params(case, seed):
    p = dict(BASE, seed=seed)
    if case["kind"] == "rmd":
        if case["reduced"]:
            p.update(integrator=0, dt=0.01, gamma=10.0, kT=1.0, dh_prefactor=0.0, k_R=0.01)
        if case["cut"] > 0:
            p.update(r_cut_contact=case["cut"], r_cut_nb=case["cut"])
    elif case["kind"] == "zbias":
        p.update(dh_prefactor=0.0)
    elif case["kind"] in ("scps", "mean"):
        p.update(bias_mode=1, k_s=50.0, k_w=5.0)
    return p


def _cv0(case, R):
    cv = np.zeros((R, 8))
    cv[:, 1] = cv[:, 5] = cv[:, 6] = INF
    if case["kind"] == "scps":           # minima reached earlier: both ratchets pull
        cv[:, 5], cv[:, 6] = -0.2, -1.0
    return cv


def prepare(case, seed):
    dev = torch.device("cuda")
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "funnel":
        return dict(kind=kind, steps=case["steps"], step=0,
                    params=dict(FUNNEL, bias_mode=case["tube"], seed=d["seed"]),
                    xy=torch.as_tensor(d["xy"], device=dev), cv=torch.as_tensor(_cv0(case, case["n"]), device=dev),
                    path=torch.as_tensor(d["path"], device=dev) if case["tube"] else None)
    R = case.get("replicas") or case["chains"]
    own = kind in ("uneven", "zbias")    # every chain its own system and native map
    ctx = scps.Context(_params(case, d["seed"]), [len(m) for _, m, _ in d["chains"]], [c for c, _, _ in d["chains"]],
                       [m for _, m, _ in d["chains"]], [q for _, _, q in d["chains"]],
                       np.arange(R) if own else np.zeros(R, np.int32))
    for s, xyz in enumerate(d["native"]):
        ctx.set_reference_map(s, native_xyz=xyz)
    x = np.concatenate([a.ravel() for a in d["x"]]) if own else d["x"].ravel()
    x = torch.as_tensor(x, device=dev)
    st = dict(kind=kind, ctx=ctx, x=x)
    if kind == "zbias":
        z = torch.empty(R, dtype=torch.float64, device=dev)
        ctx.eval_z_and_grad(x, z)
        st.update(zm=0.7 * z, grad=case["grad"])
        x.requires_grad_(bool(case["grad"]))
        return st
    if kind in ("scps", "mean"):
        st.update(frames=torch.as_tensor(d["frames"].ravel(), device=dev), n_frames=case["frames"],
                  n_paths=len(d["success"]), success=d["success"])
        if kind == "mean":
            st.update(maps=bool(case["maps"]), s=torch.empty(R, dtype=torch.float64, device=dev),
                      w=torch.empty(R, dtype=torch.float64, device=dev))
            return st
        ctx.update_reference_from_paths(0, st.pop("frames"), st["n_paths"], st["n_frames"], st["success"])
    v = np.concatenate([a.ravel() for a in d["v"]]) if own else d["v"].ravel()
    st.update(v=torch.as_tensor(v, device=dev), cv=torch.as_tensor(_cv0(case, R), device=dev), steps=case["steps"],
              step=0)
    return st


def run(st):
    kind = st["kind"]
    if kind == "funnel":
        scps.funnel_steps(st["params"], st["xy"], st["cv"], st["steps"], step0=st["step"], mean_path=st["path"])
        st["step"] += st["steps"]
        return dict(xy=st["xy"], cv=st["cv"])
    ctx, x = st["ctx"], st["x"]
    if kind == "zbias":
        if not st["grad"]:
            z, e = scps.zbias(x, st["zm"], ctx)
            return dict(z=z.to(torch.float32), e=e.to(torch.float32))
        x.grad = None
        z, e = scps.zbias(x, st["zm"], ctx)
        (z.sum() + e.sum()).backward()
        return dict(z=z.detach().to(torch.float32), e=e.detach().to(torch.float32), grad=x.grad)
    if kind == "mean":
        maps = ctx.update_reference_from_paths(0, st["frames"], st["n_paths"], st["n_frames"], st["success"],
                                               want_maps=st["maps"])
        ctx.eval_tube(0, x, st["s"], st["w"])
        out = dict(s=st["s"].to(torch.float32), w=st["w"].to(torch.float32))
        return dict(out, maps=maps) if st["maps"] else out
    ctx.step_replicas(x, st["v"], st["cv"], st["steps"], step0=st["step"])
    st["step"] += st["steps"]
    return dict(x=x, v=st["v"], cv=st["cv"].to(torch.float32))


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
# Operations per unordered pair (an FMA counts 2; rcp, rsqrt, exp 1 each):
# contact z and gradient 43, z alone 21, Lennard-Jones and Debye-Hueckel 40,
# the two together 75 (shared geometry); per frame and pair 3 for the squared
# difference and 2 for the effective reference of the SCPS bias.
def work(case):
    kind = case["kind"]
    if kind == "funnel":
        n = case["n"]
        return dict(bytes=n * (32 + 128), flops=n * case["steps"] * (60 + (32 * case["frames"] if case["tube"] else 20)))
    if kind == "uneven":
        sizes = _sizes(case).astype(np.float64)
        pairs = float((sizes * (sizes - 1) / 2).sum())
        return dict(bytes=case["steps"] * 4 * pairs + 48 * float(sizes.sum()), flops=case["steps"] * 75 * pairs)
    if kind == "zbias":
        pairs = case["chains"] * case["n"] * (case["n"] - 1) / 2
        return dict(bytes=4 * pairs + 24 * case["chains"] * case["n"], flops=pairs * (43 if case["grad"] else 21))
    n, R = case["n"], case["replicas"]
    nc = int(np.count_nonzero(np.arange(n) % 16 < 8)) if case["heavy"] else n
    con, nb = nc * (nc - 1) / 2, max(0, (n - 2) * (n - 3) / 2)
    state = 48 * R * n
    if kind == "rmd":
        if case["cut"] > 0:
            # pairs inside the cutoff of a compact chain (one particle per lattice cell)
            near = n * min(n - 1, 4.19 * (case["cut"] / LATTICE) ** 3) / 2
            return dict(bytes=state + case["steps"] * R * (2 * near * 4 + 16 * n), flops=case["steps"] * R * 75 * near)
        nbf = 24 if case["reduced"] else 40
        return dict(bytes=state + 4 * con, flops=case["steps"] * R * (43 * con + nbf * nb - 8 * min(con, nb)))
    K = case["frames"]
    if kind == "scps":
        return dict(bytes=state + case["steps"] * 4 * K * con,
                    flops=case["steps"] * R * ((18 + 3 * K + 43 + 2 * K) * con + 32 * nb))
    return dict(bytes=12 * K * R * n + 4 * K * con, flops=R * K * 18 * con + 2 * (18 + 3 * K) * R * con)


# ---------------------------------------------------------------------------
# the same results in float64
# ---------------------------------------------------------------------------
def _contact(r2, p):
    q = r2 / p["r0_contact"] ** 2
    num = 1 + q + q * q
    den = num + q ** 3 + q ** 4
    c = num / den
    dc = (1 + 2 * q) / den - num * (1 + 2 * q + 3 * q * q + 4 * q ** 3) / den ** 2
    if p["r_cut_contact"] > 0:
        out = r2 > p["r_cut_contact"] ** 2
        c = c.masked_fill(out, 0.0)
        dc = dc.masked_fill(out, 0.0)
    return c, dc


def _philox_normals(seed, atom, rep, step):
    """[R, n, 3] standard normals (Philox4x32-10, Box-Muller in float64)."""
    m32 = 0xFFFFFFFF
    R, n = len(rep), len(atom)
    c = [atom[None, :].expand(R, n), rep[:, None].expand(R, n), torch.full((R, n), step & m32, device=atom.device),
         torch.full((R, n), step >> 32, device=atom.device)]
    k0, k1 = seed & m32, seed >> 32

    def mulhilo(a, b):
        # 32 x 32 -> 64 bits in two halves, so that nothing passes 2^63
        lo16, hi16 = b & 0xFFFF, b >> 16
        p0, p1 = a * lo16, a * hi16
        mid = p1 + (p0 >> 16)
        return mid >> 16, ((mid & 0xFFFF) << 16) | (p0 & 0xFFFF)

    for _ in range(10):
        h0, l0 = mulhilo(0xD2511F53, c[0])
        h1, l1 = mulhilo(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    u = [((w >> 9) * 2 + 1).double() * 2.0 ** -24 for w in c]
    r01, r23 = torch.sqrt(-2 * torch.log(u[0])), torch.sqrt(-2 * torch.log(u[2]))
    a1, a3 = 2 * math.pi * u[1], 2 * math.pi * u[3]
    return torch.stack([r01 * torch.cos(a1), r01 * torch.sin(a1), r23 * torch.cos(a3)], -1)


class _Exact:
    """Forces of a batch of replicas of one chain, x [R, 3, n] float64."""

    def __init__(self, p, chain, native, dev):
        self.p, self.dev = p, dev
        ci, mass, charge = chain
        self.n = len(mass)
        self.mass = torch.as_tensor(mass.astype(np.float64), device=dev)
        self.q = torch.as_tensor(charge.astype(np.float64), device=dev)
        self.on = torch.zeros(self.n, dtype=torch.bool, device=dev)
        self.on[torch.as_tensor(ci.astype(np.int64), device=dev)] = True
        self.idx = torch.arange(self.n, device=dev)
        self.native = torch.as_tensor(native, device=dev)

    def rows(self, R):
        per = max(1, min(self.n, int(2.5e7 // (R * self.n))))
        return [slice(a, min(a + per, self.n)) for a in range(0, self.n, per)]

    def geometry(self, x, sl):
        d = x[:, :, sl, None] - x[:, :, None, :]             # [R, 3, rows, n]
        return d, (d * d).sum(1)

    def mask(self, sl):
        """(contact pairs, nonbonded pairs) of rows sl."""
        sep = (self.idx[sl, None] - self.idx[None, :]).abs()
        con = self.on[sl, None] & self.on[None, :] & (sep > 0)
        return con, sep > self.p["nb_excl"]

    def ref(self, sl):
        d, r2 = self.geometry(self.native[None], sl)
        return _contact(r2, self.p)[0][0]

    def nonbonded(self, x):
        p, F = self.p, torch.zeros_like(x)
        for sl in self.rows(len(x)):
            d, r2 = self.geometry(x, sl)
            _, nb = self.mask(sl)
            nb = nb[None] & ((r2 <= p["r_cut_nb"] ** 2) if p["r_cut_nb"] > 0 else True)
            r2 = torch.where(nb, r2, torch.ones((), dtype=r2.dtype, device=r2.device))
            s6 = (p["lj_sigma"] ** 2 / r2) ** 3
            f = 24 * p["lj_eps"] * (2 * s6 * s6 - s6)
            if p["dh_prefactor"]:
                r = torch.sqrt(r2)
                f = f + p["dh_prefactor"] * self.q[sl, None] * self.q[None, :] * torch.exp(-p["dh_kappa"] * r) * (
                    p["dh_kappa"] + 1 / r)
            F[:, :, sl] = (torch.where(nb, f / r2, 0.0)[:, None] * d).sum(-1)
        b = x[:, :, 1:] - x[:, :, :-1]
        r = torch.sqrt((b * b).sum(1, keepdim=True))
        g = p["k_bond"] * (r - p["r_bond"]) / r * b
        F[:, :, :-1] += g
        F[:, :, 1:] -= g
        return F

    def z_grad(self, x, grad=True):
        p = self.p
        z, G = torch.zeros(len(x), dtype=x.dtype, device=x.device), torch.zeros_like(x)
        for sl in self.rows(len(x)):
            d, r2 = self.geometry(x, sl)
            con, _ = self.mask(sl)
            c, dc = _contact(r2, p)
            u = torch.where(con, c - self.ref(sl), 0.0)
            z += 0.5 * (u * u).sum((1, 2))
            if grad:
                G[:, :, sl] = (4 / p["r0_contact"] ** 2) * ((u * dc)[:, None] * d).sum(-1)
        return z, G

    def stack(self, frames, succ):
        """The mean maps as [K, n, n] (float64), over the successful paths."""
        keep = torch.as_tensor(frames[:, np.nonzero(succ)[0]], device=self.dev)
        S = torch.zeros(len(frames), self.n, self.n, dtype=torch.float64, device=self.dev)
        for k in range(len(frames)):
            f = keep[k].double()
            for sl in self.rows(len(f)):
                _, r2 = self.geometry(f, sl)
                S[k, sl] = _contact(r2, self.p)[0].mean(0)
        con = self.mask(slice(0, self.n))[0]
        return S.mul_(con)

    def z0(self):
        return float(sum(0.5 * (self.ref(sl) ** 2 * self.mask(sl)[0]).sum() for sl in self.rows(1)))

    def tube(self, x, S, Z0, grad=None):
        """d [R, K], s, w, p of every replica against the stack."""
        K, lam = len(S), self.p["lam"]
        con = self.mask(slice(0, self.n))[0]
        d = torch.zeros(len(x), K, dtype=torch.float64, device=self.dev)
        SS = torch.stack([(m * m).sum() for m in S])
        for r in range(len(x)):
            cc, dot = 0.0, torch.zeros(K, dtype=torch.float64, device=self.dev)
            for sl in self.rows(1):
                _, r2 = self.geometry(x[r:r + 1], sl)
                c = _contact(r2[0], self.p)[0] * con[sl]
                cc = cc + (c * c).sum()
                dot += S[:, sl].reshape(K, -1) @ c.reshape(-1)
            d[r] = 0.5 * (cc - 2 * dot + SS) / Z0
        a = (-lam * d).amax(1, keepdim=True)
        e = torch.exp(-lam * d - a)
        pk = e / e.sum(1, keepdim=True)
        k = torch.arange(K, dtype=torch.float64, device=self.dev)
        kbar = (pk * k).sum(1)
        return 1 - kbar / (K - 1), -(a[:, 0] + torch.log(e.sum(1))) / lam, pk, kbar, k

    def tube_force(self, x, S, Z0, cv):
        p = self.p
        s, w, pk, kbar, k = self.tube(x, S, Z0)
        sm, wm = torch.minimum(cv[:, 5], s), torch.minimum(cv[:, 6], w)
        ds, dw = s - sm, w - wm
        K = len(S)
        ck = pk * (p["k_s"] * ds[:, None] * (p["lam"] / (K - 1)) * (k[None] - kbar[:, None]) + p["k_w"] * dw[:, None])
        ck = ck / Z0
        F = torch.zeros_like(x)
        con = self.mask(slice(0, self.n))[0]
        for r in range(len(x)):
            for sl in self.rows(1):
                d, r2 = self.geometry(x[r:r + 1], sl)
                c, dc = _contact(r2[0], p)
                E = (ck[r] @ S[:, sl].reshape(K, -1)).reshape(c.shape)
                u = torch.where(con[sl], (ck[r].sum() * c - E) * dc, 0.0)
                F[r, :, sl] = -(4 / p["r0_contact"] ** 2) * (u[None] * d[0]).sum(-1)
        cv[:, 3], cv[:, 4], cv[:, 5], cv[:, 6] = s, w, sm, wm
        cv[:, 2] = 0.5 * p["k_s"] * ds ** 2 + 0.5 * p["k_w"] * dw ** 2
        return F

    def steps(self, x, v, cv, n_steps, rep0, S=None):
        p = self.p
        rep = torch.arange(rep0, rep0 + len(x), device=self.dev)
        Z0 = self.z0() if S is not None else 0.0
        for m in range(n_steps):
            F = self.nonbonded(x)
            if S is not None:
                Fb = self.tube_force(x, S, Z0, cv)
            else:
                z, G = self.z_grad(x)
                cv[:, 0] = z
                cv[:, 1] = torch.minimum(cv[:, 1], z)
                dz = z - cv[:, 1]
                cv[:, 2] = 0.5 * p["k_R"] * dz ** 2
                Fb = -p["k_R"] * dz[:, None, None] * G
            cv[:, 7] += p["dt"] / p["gamma"] * (Fb * Fb / self.mass).sum((1, 2))
            F = F + Fb
            g = _philox_normals(p["seed"], self.idx, rep, m).transpose(1, 2)
            if p["integrator"] == 0:
                mob = p["dt"] / (self.mass * p["gamma"])
                x = x + mob * F + torch.sqrt(2 * p["kT"] * mob) * g
            else:
                c1 = math.exp(-p["gamma"] * p["dt"])
                v = v + p["dt"] * F / self.mass
                x = x + 0.5 * p["dt"] * v
                v = c1 * v + torch.sqrt((1 - c1 * c1) * p["kT"] / self.mass) * g
                x = x + 0.5 * p["dt"] * v
        return x, v, cv


def _exact_funnel(case, d, dev):
    P = FUNNEL
    X = torch.as_tensor(d["xy"], device=dev)
    cv = torch.as_tensor(_cv0(case, case["n"]), device=dev)
    path = torch.as_tensor(d["path"], device=dev)
    D, lam, K = P["mob_dt"], P["lam"], case["frames"]
    ids = torch.arange(case["n"], device=dev)
    k = torch.arange(K, dtype=torch.float64, device=dev)
    for m in range(case["steps"]):
        r2 = (X * X).sum(1)
        dx = X - torch.tensor([P["xm"], P["ym"]], dtype=torch.float64, device=dev)
        gr = 4 * P["w"] ** 2 * r2 + 4 * P["A1"] * P["s1"] ** 2 / (r2 + P["s1"] ** 2) ** 3 - 4 * P["A2"] * P[
            "s2"] ** 2 / (r2 + P["s2"] ** 2) ** 3
        g3 = 4 * P["A3"] * P["s3"] ** 2 / ((dx * dx).sum(1) + P["s3"] ** 2) ** 3
        F = -(gr[:, None] * X + g3[:, None] * dx)
        if case["tube"]:
            e = X[:, None] - path[None]
            pk = torch.softmax(-lam * (e * e).sum(-1), 1)
            w = -torch.logsumexp(-lam * (e * e).sum(-1), 1) / lam
            kbar = (pk * k).sum(1)
            s = 1 - kbar / (K - 1)
            gs = (lam / (K - 1)) * (pk * (k[None] - kbar[:, None]))[:, :, None].mul(2 * e).sum(1)
            gw = (pk[:, :, None] * 2 * e).sum(1)
            cv[:, 3], cv[:, 4] = s, w
            cv[:, 5], cv[:, 6] = torch.minimum(cv[:, 5], s), torch.minimum(cv[:, 6], w)
            ds, dw = s - cv[:, 5], w - cv[:, 6]
            Fb = -P["k_s"] * ds[:, None] * gs - P["k_w"] * dw[:, None] * gw
            cv[:, 2] = 0.5 * P["k_s"] * ds ** 2 + 0.5 * P["k_w"] * dw ** 2
        else:
            z = torch.sqrt(r2)
            cv[:, 0], cv[:, 1] = z, torch.minimum(cv[:, 1], z)
            dz = z - cv[:, 1]
            Fb = -P["k_R"] * (dz / z)[:, None] * X
            cv[:, 2] = 0.5 * P["k_R"] * dz ** 2
        cv[:, 7] += D * (Fb * Fb).sum(1)
        g = _philox_normals(d["seed"], torch.zeros(1, dtype=torch.int64, device=dev), ids, m)[:, 0, :2]
        X = X + D * (F + Fb) + math.sqrt(2 * P["kT"] * D) * g
    return dict(xy=X, cv=cv)


def exact(case, seed):
    dev = device()
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "funnel":
        return _exact_funnel(case, d, dev)
    p = _params(case, d["seed"])

    def state(a):
        return torch.as_tensor(np.asarray(a), device=dev).double()

    if kind in ("uneven", "zbias"):
        out = []
        for r in range(len(d["chains"])):
            ex = _Exact(p, d["chains"][r], d["native"][r], dev)
            x = state(d["x"][r])[None]
            if kind == "zbias":
                z, G = ex.z_grad(x, bool(case["grad"]))
                dz = z - 0.7 * z
                out.append((z, 0.5 * p["k_R"] * dz ** 2, (1 + p["k_R"] * dz)[:, None, None] * G))
            else:
                cv = torch.as_tensor(_cv0(case, 1), device=dev)
                out.append(ex.steps(x, state(d["v"][r])[None], cv, case["steps"], r))
        flat = [torch.cat([o[k].reshape(-1) for o in out]) for k in range(3)]
        if kind == "zbias":
            return dict(z=flat[0], e=flat[1], grad=flat[2]) if case["grad"] else dict(z=flat[0], e=flat[1])
        return dict(x=flat[0], v=flat[1], cv=flat[2].reshape(-1, 8))
    ex = _Exact(p, d["chains"][0], d["native"][0], dev)
    x = state(d["x"])
    if kind == "mean":
        S = ex.stack(d["frames"], d["success"])
        s, w, *_ = ex.tube(x, S, ex.z0())
        if not case["maps"]:
            return dict(s=s, w=w)
        ci = torch.as_tensor(d["chains"][0][0].astype(np.int64), device=dev)
        a, b = torch.triu_indices(len(ci), len(ci), 1, device=dev)
        return dict(s=s, w=w, maps=S[:, ci[a], ci[b]])
    S = ex.stack(d["frames"], d["success"]) if kind == "scps" else None
    cv = torch.as_tensor(_cv0(case, len(x)), device=dev)
    x, v, cv = ex.steps(x, state(d["v"]), cv, case["steps"], 0, S)
    return dict(x=x.reshape(-1), v=v.reshape(-1), cv=cv)
