"""The work that users of libpfmm have it do, as cases that can be timed and checked.

A case names one call (or one step of a fit) and its sizes; ``prepare`` makes
the inputs and the plan on the GPU, ``run`` is one pass through the public
entry points, and ``exact`` gives the same outputs in FP64 by plain torch: the
tree's own sums (Eqs. 5-7 and the 27-leaf near zone) with every block
convolution done by an FP64 FFT on its doubled grid, which is exact up to
rounding, and gradients by automatic differentiation of that.
"""
import math
import random

import numpy as np
import torch

from paper_2011_07099_amd.pfmm import Batch, Plan

DEV = "cuda"
# How a plan sums its zones: the options a user passes to Plan.
ROUTES = {
    "plain": {},                                         # the defaults: FP32, direct near zone, GEMM zones
    "split": {"precision": "bf16x3"},                    # the same on the BF16 matrix cores
    "fast": {"near": "fft", "m2l": "spectral"},          # transforms: the benchmark's routes
    "f64": {"precision": "fp64"},                        # FP64 throughout, FP64 arrays
}


def _case(name, kind, N, L, p, route="plain", accel="none", isolated=False, zones_fp32=False,
          fields=1, sigma=1.0):
    c = {"kind": kind, "N": N, "L": L, "p": p, "route": route, "accel": accel,
         "isolated": isolated, "zones_fp32": zones_fp32, "fields": fields,
         "sigma": sigma}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a small box solved on its own, as in a time step of a small run or the smoke check:
        # a call is a chain of short launches, so latency and their number count
        _case("solve_32_p4", "solve", 32, 3, 4, "fast"),
        # a user who sets no option, an odd gridlet (p = 7) and accelerations by differences
        _case("solve_64_p7_plain", "solve", 64, 3, 7, "plain", "fd4"),
        # the middle of the batch workload's sizes, one field on its own
        _case("solve_128_p6", "solve", 128, 3, 6, "fast", "fd4"),
        # the benchmark: 256^3, four levels, p = 8, FP32 leaf columns
        _case("solve_256_p8", "solve", 256, 4, 8, "fast", zones_fp32=True, sigma=2.0),
        # the same box on the matrix cores (direct near zone, GEMM zones)
        _case("solve_256_p8_split", "solve", 256, 4, 8, "split", sigma=2.0),
        # the largest box that is in everyday use, five levels
        _case("solve_512_p8", "solve", 512, 5, 8, "fast", sigma=2.0),
        # the force-error measurement: point sources, accelerations from the expansion
        _case("force_128_p8", "force", 128, 3, 8, "plain", "expansion"),
        # a reference solve in FP64
        _case("solve_64_p8_f64", "solve", 64, 3, 8, "f64"),
        # many independent boxes of mixed sizes in one graph launch
        _case("batch_32_fields", "batch", 128, 3, 8, "fast", fields=32),
        # one gradient of the grid-valued tables' fit, a large training field (16^3-cell leaves)
        _case("fit_table_128_p4", "table", 128, 3, 4),
        # one gradient of the network's fit over two fields of the training workload's size
        _case("fit_net_64_p4", "net", 64, 3, 4, fields=2),
        # one gradient of the fit of G_* used everywhere, at the fit's mesh and depth
        _case("fit_gstar_64_p2", "gstar", 64, 4, 2),
    ]


def draw(rng):
    """One more case, its density's contrast spread like the batch workload's."""
    c = _draw(rng)
    return dict(c, sigma=round(rng.uniform(0.5, 1.2 if c["kind"] != "batch" else 2.0), 3))


def _draw(rng):
    """Leaves are 2 to 16 cells wide, gridlets 2 to 9 nodes; the
    doubled-grid and spectral routes take the widths and gridlets they serve.
    Fits stay at low orders and differenced accelerations at N <= 128 (not
    split): beyond that the FMM-vs-PM residual and the differences of the
    potential are of the size of its FP32 rounding."""
    kind = rng.choice(["solve"] * 6 + ["force", "force", "batch", "table", "net", "gstar"])
    if kind == "solve":
        route = rng.choice(["fast", "fast", "fast", "plain", "plain", "split", "f64"])
        accel = rng.choice(["none", "fd4"])
        if route == "fast":
            p, s = rng.choice([4, 6, 8]), rng.choice([4, 8, 16])
            L = rng.choice([l for l in (2, 3, 4, 5) if 16 <= s << l <= 256])
            z = L == 4 and rng.random() < 0.5
            accel = accel if s << L <= 128 and not z else "none"
            return _case(None, kind, s << L, L, p, route, accel, rng.random() < 0.1, z)
        if route == "split":
            s = rng.choice([8, 16])
            L = rng.choice([l for l in (2, 3, 4) if s << l <= 128])
            return _case(None, kind, s << L, L, 8, route)
        s = rng.choice([2, 4, 8, 16])
        most = 64 if route == "f64" else 128
        L = rng.choice([l for l in (2, 3, 4) if s << l <= most])
        p = rng.randrange(2, 10 if route == "plain" else 9)
        return _case(None, kind, s << L, L, p, route, accel, rng.random() < 0.1)
    if kind == "force":
        s, p = rng.choice([4, 8, 16]), rng.choice([4, 5, 6, 8])
        L = rng.choice([l for l in (2, 3) if s << l <= 128])
        route = "plain" if p == 5 else rng.choice(["plain", "fast"])
        return _case(None, kind, s << L, L, p, route, "expansion", rng.random() < 0.5)
    if kind == "batch":
        return _case(None, kind, rng.choice([32, 64, 128]), 3, rng.choice([4, 6, 8]), "fast",
                     fields=rng.randrange(3, 32))
    if kind == "gstar":
        N, L = rng.choice([(16, 2), (32, 2), (32, 3), (64, 4)])
        return _case(None, kind, N, L, 2, fields=1 if N == 64 else rng.randrange(1, 4))
    N, L, p = rng.choice([(32, 2, 3), (64, 2, 3), (64, 3, 3), (64, 3, 4), (128, 3, 3), (128, 3, 4)])
    p = min(p, 3) if kind == "table" and N == 64 else p
    return _case(None, kind, N, L, p, fields=1 if N == 128 else rng.randrange(1, 5))


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(1 + int(seed))


def _lognormal(N, gen, alpha=2.0, sigma=1.0):
    """exp(delta) - mean, delta a Gaussian field with P(k) ~ k^-alpha."""
    w = torch.fft.rfftn(torch.randn((N, N, N), generator=gen, device=DEV))
    k = torch.fft.fftfreq(N, d=1.0 / N, device=DEV)
    kz = torch.arange(N // 2 + 1, device=DEV, dtype=k.dtype)
    k2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + kz[None, None, :] ** 2
    k2[0, 0, 0] = 1.0
    w *= k2 ** (-0.25 * alpha)
    w[0, 0, 0] = 0.0
    d = torch.fft.irfftn(w, s=(N, N, N))
    rho = torch.exp(sigma / d.std() * d)
    return (rho - rho.mean()).contiguous()


def _points(N, gen, isolated):
    """Ten sources of mass 1/8 in single cells (not mean-subtracted when isolated)."""
    at = torch.randint(0, N ** 3, (10,), generator=gen, device=DEV)
    rho = torch.zeros(N ** 3, device=DEV)
    rho.index_add_(0, at, torch.full((10,), float(N) ** 3 / 8.0, device=DEV))
    rho = rho.reshape(N, N, N)
    return rho if isolated else rho - rho.mean()


def _members(case):
    """(N, p) of each field: a single solve, or a batch's mix up to the case's sizes."""
    if case["kind"] != "batch":
        return [(case["N"], case["p"])] * case["fields"]
    r = random.Random(1000 * case["N"] + 10 * case["p"] + case["fields"])
    Ns = [n for n in (32, 64, 128) if n <= case["N"]]
    ps = [q for q in (4, 6, 8) if q <= case["p"]]
    return [(r.choice(Ns), r.choice(ps)) for _ in range(case["fields"])]


def _densities(case, seed):
    gen = _gen(seed)
    if case["kind"] == "force":
        return [_points(case["N"], gen, case["isolated"])]
    rhos = [_lognormal(n, gen, 1.5 if n >= 256 else 2.0, case["sigma"]) for n, _ in _members(case)]
    return [r.double() for r in rhos] if case["route"] == "f64" else rhos


def _green(case):
    """(kind, (a1, a2)) of the plan's G."""
    if case["isolated"]:
        return "X", None
    return ("S", (-0.125, 0.0)) if case["kind"] == "force" else ("S1", (-0.125, 0.0))


def _orbits(n):
    return n * (n + 1) * (n + 2) // 6


def _parameters(case, seed):
    """The fit's current parameters: table corrections, network weights or G_*'s."""
    r = np.random.default_rng(seed)
    if case["kind"] == "table":
        n = (case["L"] - 1) * _orbits(4 * case["p"])
        return (1e-6 * r.standard_normal(n)).astype(np.float32)
    if case["kind"] == "gstar":
        return (1e-4 * r.standard_normal(_orbits(case["N"] // 2 + 1))).astype(np.float32)
    w1 = 4.0 * r.standard_normal((64, 8))
    b1 = -np.sum(w1 * r.uniform(size=(64, 8)), axis=1)
    w2 = np.sqrt(2.0 / 64) * r.standard_normal((64, 64))
    w3 = 0.02 * r.standard_normal(64)
    return np.concatenate([w1.ravel(), b1, w2.ravel(), np.zeros(64), w3, [0.0]]).astype(np.float32)


def _target(rho):
    """PM with G_S1 (the exact periodic convolution), as training holds it."""
    N = rho.shape[0]
    lat = _green_grid("S1", (-0.125, 0.0), _folded(N) / N, 1.0 / N)
    return _pm(rho.double(), lat).float()


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    rhos = _densities(case, seed)
    green, _ = _green(case)
    kw = dict(ROUTES[case["route"]])
    if case["isolated"]:
        kw["isolated"] = True
    if case["zones_fp32"]:
        kw["zones_fp32"] = True
    if case["kind"] == "force":  # zones in FP64 at every level, as the error measurement sets them
        kw.update(accel="expansion", fp64_levels=case["L"] - 1)
        if green == "S":
            kw["a1"] = -0.125
    st = {"case": case, "rhos": rhos}
    if case["kind"] == "batch":
        st["plans"] = [Plan(n, case["L"], p, green, **kw) for n, p in _members(case)]
        st["phis"] = [torch.empty_like(r) for r in rhos]
        st["batch"] = Batch(st["plans"], rhos, st["phis"])
        return st
    plan = st["plan"] = Plan(case["N"], case["L"], case["p"], green, **kw)
    if case["kind"] in ("solve", "force"):
        st["phi"] = torch.empty_like(rhos[0])
        st["acc"] = None
        if case["accel"] != "none":
            st["acc"] = torch.empty((3,) + tuple(rhos[0].shape), dtype=rhos[0].dtype, device=DEV)
        return st
    st["par"] = _parameters(case, seed)
    if case["kind"] == "gstar":
        plan.set_gstar(st["par"])
        return st
    st["targets"] = [_target(r) for r in rhos]
    if case["kind"] == "table":
        plan.table_train_begin(1e-6)
    return st


def run(st):
    kind = st["case"]["kind"]
    if kind == "batch":
        st["batch"].solve()
        return st["phis"]
    plan = st["plan"]
    if kind in ("solve", "force"):
        plan.solve(st["rhos"][0], st["phi"], st["acc"])
        return {"phi": st["phi"]} if st["acc"] is None else {"phi": st["phi"], "acc": st["acc"]}
    if kind == "gstar":     # one gradient of the conjugate-gradient fit
        plan.set_gstar(st["par"])
        loss = [plan.gstar_accumulate(r) for r in st["rhos"]]
        return {"loss": loss, "grad": plan.gstar_grad()}
    if kind == "table":
        plan.set_table(st["par"])
        loss = [plan.train_accumulate(r, t) for r, t in zip(st["rhos"], st["targets"])]
        return {"loss": loss, "grad": plan.table_grad()}
    plan.train_begin(st["par"], 1e-3)
    loss = [plan.train_accumulate(r, t) for r, t in zip(st["rhos"], st["targets"])]
    return {"loss": loss, "grad": plan.learned_grads(2)[1]}


def _solve_flops(N, L, p, kernels=1):
    """The sums per frequency of the doubled blocks and their transforms, the
    cheapest form known: 27 and 189 complex multiply-adds, 5 n log2 n an FFT."""
    s = N >> L

    def blocks(n, q, offs, k):
        freq = 4 * q * q * (q + 1)
        fft = 2.5 * (2 * q) ** 3 * math.log2((2 * q) ** 3) if q > 1 else 8.0
        return n * (8.0 * freq * offs * k + (1 + k) * fft)

    f = blocks(8 ** L, s, 27, kernels) + blocks(64, p, 37, 1)
    f += sum(blocks(8 ** l, p, 189, 1) for l in range(3, L + 1))
    f += 2 * 8 ** L * 2 * (s ** 3 * p + s * s * p * p + s * p ** 3)       # P2M, L2P
    return f + 2 * sum(8 ** l * 28 * p ** 4 for l in range(2, L))         # M2M, L2L


def work(case):
    """Densities (and targets) in, potentials, accelerations or gradients out;
    an adjoint sweep and table gradient cost about what the solve does."""
    L, kind = case["L"], case["kind"]
    b = f = 0.0
    for N, p in _members(case):
        n3 = float(N) ** 3
        if kind in ("solve", "force", "batch"):
            w = 8 if case["route"] == "f64" else 4
            b += n3 * w * (2 + (0 if case["accel"] == "none" else 3))
            f += _solve_flops(N, L, p, 4 if case["accel"] == "expansion" else 1)
            f += 24 * n3 if case["accel"] == "fd4" else 0
        else:
            b += n3 * 4 * (1 if kind == "gstar" else 2)
            f += 2 * _solve_flops(N, L, p)
            if kind == "gstar":     # PM and its correlation: four FFTs of the mesh
                f += 4 * 2.5 * n3 * math.log2(n3)
    if kind == "table":
        b += 8.0 * (L - 1) * _orbits(4 * case["p"])
    if kind == "gstar":
        b += 8.0 * _orbits(case["N"] // 2 + 1)
    if kind == "net":
        b += 8.0 * 4801
        f += (2 + 4 * case["fields"]) * 4801.0 * (L - 1) * _orbits(4 * case["p"])
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same outputs in FP64 (plain torch)
# ---------------------------------------------------------------------------

def _f64(x):
    return torch.as_tensor(x, dtype=torch.float64, device=DEV)


def _folded(N):
    j = torch.arange(N, device=DEV, dtype=torch.float64)
    return torch.where(j < N // 2, j, j - N)


def _green_grid(kind, a, x, h, free=False):
    """G on the product grid x^3 of separations; G(0) is the cube self value for
    h > 0. Kinds S, S1: the map of Sec. 3; X: nearest image; free: no images."""
    if kind == "X":
        v = x if free else x - torch.round(x)
    else:
        base = torch.sin(math.pi * x) / math.pi
        v = base + sum(ak * (torch.sin(m * math.pi * x) / (m * math.pi) - base)
                       for ak, m in zip(a, (3, 5)))
    r = torch.sqrt(v[:, None, None] ** 2 + v[None, :, None] ** 2 + v[None, None, :] ** 2)
    x0 = x == 0
    zero = x0[:, None, None] & x0[None, :, None] & x0[None, None, :]
    g = -1.0 / (4 * math.pi * torch.where(zero, torch.ones_like(r), r))
    r3 = math.sqrt(3.0)
    c0 = 3.0 * math.log((r3 + 1) / (r3 - 1)) - math.pi / 2
    return torch.where(zero, torch.full_like(g, -c0 / (4 * math.pi * h) if h else 0.0), g)


def _weights(p, v, deriv=False):
    """W[a, c]: Lagrange basis a of the gridlet nodes at v_c (or its derivative)."""
    t = np.arange(p) + 0.5 - 0.5 * p
    V = t[None, :] ** np.arange(p)[:, None]
    n = np.arange(p)[:, None]
    S = n * v[None, :] ** np.maximum(n - 1, 0) if deriv else v[None, :] ** n
    return _f64(np.linalg.solve(V, S))


def _apply3(ops, x):
    """Contract the last three axes of x with ops[i][out, in]."""
    for i, op in enumerate(ops):
        x = torch.movedim(torch.tensordot(x, op, dims=([x.dim() - 3 + i], [1])), -1, x.dim() - 3 + i)
    return x


def _blocks(X, tab, q, spans, keep, periodic):
    """Y[t][a] = sum_d sum_a' tab[a - a' - q d] X[t + d][a'] over the offsets d
    (|d_i| <= 3) that keep(d) holds, for the targets whose class has them:
    spans(d_i) gives the first target and step per axis, or None."""
    n, C = X.shape[0], (tab.shape[0] - 1) // 2
    m = torch.arange(2 * q, device=DEV)
    m = torch.where(m < q, m, m - 2 * q)
    Xh = torch.fft.rfftn(X, s=(2 * q,) * 3, dim=(3, 4, 5))
    out = torch.zeros_like(Xh)
    rng = [d for d in range(-3, 4) if spans(d) is not None]

    def axis(d):
        t = torch.arange(spans(d)[0], n, spans(d)[1], device=DEV)
        if not periodic:
            t = t[(t + d >= 0) & (t + d < n)]
        return t, (t + d) % n

    idx = {d: (m - q * d + C).clamp(0, 2 * C) for d in rng}
    live = (m > -q).double()
    live = live[:, None, None] * live[None, :, None] * live[None, None, :]
    for d in [(a, b, c) for a in rng for b in rng for c in rng if keep((a, b, c))]:
        K = tab[idx[d[0]][:, None, None], idx[d[1]][None, :, None], idx[d[2]][None, None, :]]
        Kh = torch.fft.rfftn(K * live, dim=(0, 1, 2))
        (tx, ux), (ty, uy), (tz, uz) = (axis(v) for v in d)
        if min(len(tx), len(ty), len(tz)) == 0:
            continue
        T = (tx[:, None, None], ty[None, :, None], tz[None, None, :])
        out[T] = out[T] + Kh * Xh[ux[:, None, None], uy[None, :, None], uz[None, None, :]]
    del Xh
    return torch.fft.irfftn(out, s=(2 * q,) * 3, dim=(3, 4, 5))[..., :q, :q, :q]


def _mesh(b):
    n, s = b.shape[0], b.shape[3]
    return b.permute(0, 3, 1, 4, 2, 5).reshape(n * s, n * s, n * s)


def _tables(case):
    N, L, p = case["N"], case["L"], case["p"]
    kind, a = _green(case)
    j = torch.arange(-(4 * p - 1), 4 * p, device=DEV, dtype=torch.float64)
    tabs = {l: _green_grid(kind, a, j / (2 ** l * p), 0.0, case["isolated"]) for l in range(2, L + 1)}
    c = 2 * (N >> L) - 1
    j = torch.arange(-c - 2, c + 3, device=DEV, dtype=torch.float64)
    wide = _green_grid(kind, a, j / N, 1.0 / N, case["isolated"])
    return tabs, wide


def _fmm(rho, case, tabs, near, periodic):
    """(potential, leaf locals, cell masses by leaf)."""
    N, L, p = rho.shape[0], case["L"], case["p"]
    s, n = N >> L, 2 ** L
    mb = (rho / float(N) ** 3).reshape(n, s, n, s, n, s).permute(0, 2, 4, 1, 3, 5)
    A = _weights(p, (np.arange(s) + 0.5 - 0.5 * s) * (p / s))
    T = [_weights(p, (o - 0.5) * 0.5 * p + 0.5 * (np.arange(p) + 0.5 - 0.5 * p)) for o in (0, 1)]
    oct_ = [(x, y, z) for x in (0, 1) for y in (0, 1) for z in (0, 1)]
    M = {L: _apply3([A] * 3, mb)}
    for l in range(L - 1, 1, -1):
        M[l] = sum(_apply3([T[i] for i in o], M[l + 1][o[0]::2, o[1]::2, o[2]::2]) for o in oct_)
    far = lambda d: max(abs(v) for v in d) > 1  # noqa: E731
    every = lambda d: (0, 1)  # noqa: E731
    classes = lambda d: {3: (0, 2), -3: (1, 2)}.get(d, (0, 1))  # noqa: E731
    two = lambda d: (0, 1) if -2 <= d <= 1 else None  # noqa: E731
    Phi = _blocks(M[2], tabs[2], p, two if periodic else every, far, periodic)
    for l in range(3, L + 1):
        out = _blocks(M[l], tabs[l], p, classes, far, periodic)
        up = torch.zeros_like(out)
        for o in oct_:
            up[o[0]::2, o[1]::2, o[2]::2] = _apply3([T[i].T for i in o], Phi)
        Phi = out + up
    phi = _apply3([A.T] * 3, Phi) + _near(mb, near, periodic)
    return _mesh(phi), Phi, mb


def _near(mb, tab, periodic):
    return _blocks(mb, tab, mb.shape[3], lambda d: (0, 1) if abs(d) <= 1 else None,
                   lambda d: True, periodic)


def _fd4(phi):
    N = phi.shape[0]
    r = lambda k, i: torch.roll(phi, -k, i)  # noqa: E731
    return torch.stack([-N * (8 * (r(1, i) - r(-1, i)) - (r(2, i) - r(-2, i))) / 12 for i in range(3)])


def _pm(rho, lat):
    N = rho.shape[0]
    f = torch.fft.rfftn(rho) * torch.fft.rfftn(lat)
    return torch.fft.irfftn(f, s=(N, N, N)) / float(N) ** 3


def _expansion_accel(case, Phi, mb, wide):
    N, L, p = case["N"], case["L"], case["p"]
    s, c = N >> L, wide.shape[0] - 4
    v = (np.arange(s) + 0.5 - 0.5 * s) * (p / s)
    A, D = _weights(p, v), _weights(p, v, deriv=True)
    out = []
    for ax in range(3):
        sh = lambda k: wide[tuple(slice(2 + (k if i == ax else 0), 2 + (k if i == ax else 0) + c) for i in range(3))]  # noqa: E731,E501
        ker = -N * (8 * (sh(1) - sh(-1)) - (sh(2) - sh(-2))) / 12
        far = -(2 ** L * p) * _apply3([(D if i == ax else A).T for i in range(3)], Phi)
        out.append(_mesh(far + _near(mb, ker, not case["isolated"])))
    return torch.stack(out)


def _orbit(u):
    """Index of the sorted triple of |components| u (three broadcastable tensors)."""
    t = torch.sort(torch.stack(torch.broadcast_tensors(*u), -1), -1).values
    c, b, a = t[..., 0], t[..., 1], t[..., 2]
    return a * (a + 1) * (a + 2) // 6 + b * (b + 1) // 2 + c


def _cube(u):
    return u[:, None, None], u[None, :, None], u[None, None, :]


def _features(p, L):
    K = 4 * p
    rows = [(a, b, c) for a in range(K) for b in range(a + 1) for c in range(b + 1)]
    u = _f64(rows)
    x = torch.cat([u / K, (u % p) / p], 1)
    one = torch.ones((len(rows), 1), device=DEV, dtype=torch.float64)
    return torch.cat([torch.cat([x, one * (l / 8.0), one * (p / 10.0)], 1) for l in range(2, L + 1)])


def _network(th, x):
    w1, b1 = th[:512].reshape(64, 8), th[512:576]
    w2, b2 = th[576:4672].reshape(64, 64), th[4672:4736]
    act = torch.nn.functional.silu
    h = act(act(x @ w1.T + b1) @ w2.T + b2)
    return 1e-4 * (h @ th[4736:4800] + th[4800])


def _loss(phi, t):
    r = phi - t
    r = r - r.mean()
    return (r * r).sum() / ((t - t.mean()) ** 2).sum()


def _exact_fit(case, seed):
    N, L, p, kind = case["N"], case["L"], case["p"], case["kind"]
    par = _f64(_parameters(case, seed)).requires_grad_(True)
    tabs, wide = _tables(case)
    near = wide[2:-2, 2:-2, 2:-2]
    losses = []
    for rho in _densities(case, seed):
        t = None if kind == "gstar" else _target(rho).double()
        if kind == "gstar":
            fold = lambda j: torch.minimum(j % N, N - j % N)  # noqa: E731
            j = torch.arange(-(4 * p - 1), 4 * p, device=DEV)
            cur = {l: g * (1 + par[_orbit(_cube(fold(j * ((N >> l) // p))))]) for l, g in tabs.items()}
            c = near.shape[0] // 2
            nr = near * (1 + par[_orbit(_cube(fold(torch.arange(-c, c + 1, device=DEV))))])
            lat = _green_grid("S1", (-0.125, 0.0), _folded(N) / N, 1.0 / N)
            lat = lat * (1 + par[_orbit(_cube(fold(torch.arange(N, device=DEV))))])
            t = _pm(rho.double(), lat)
        else:
            j = torch.arange(-(4 * p - 1), 4 * p, device=DEV).abs()
            delta = (_network(par, _features(p, L)) if kind == "net" else par).reshape(L - 1, -1)
            cur = {l: g * (1 + delta[l - 2][_orbit(_cube(j))]) for l, g in tabs.items()}
            nr = near
        loss = _loss(_fmm(rho.double(), case, cur, nr, True)[0], t)
        loss.backward()
        losses.append(loss.item())
    return {"loss": losses, "grad": par.grad}


def exact(case, seed):
    if case["kind"] in ("table", "net", "gstar"):
        return _exact_fit(case, seed)
    out = []
    for rho, (N, p) in zip(_densities(case, seed), _members(case)):
        sub = dict(case, N=N, p=p)
        tabs, wide = _tables(sub)
        phi, Phi, mb = _fmm(rho.double(), sub, tabs, wide[2:-2, 2:-2, 2:-2], not case["isolated"])
        out.append(phi)
    if case["kind"] == "batch":
        return out
    if case["accel"] == "none":
        return {"phi": phi}
    return {"phi": phi, "acc": _fd4(phi) if case["accel"] == "fd4" else _expansion_accel(case, Phi, mb, wide)}
