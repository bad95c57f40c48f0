"""The work that a program using the library has it do, as timed cases.

Every case goes through the public binding (paper_2509_01855_amd.birk) with the plan, the
Jacobians and the output buffers that such a program keeps.  ``op`` is the entry point:

  product   birk_apply / birk_apply_T (transpose) on one instance
  batch     birk_apply over uneven instances of one plan
  bform     birk_apply_b / birk_apply_bT
  endpoint  birk_endpoint
  fast_ax   birk_fast_ax
  precond   birk_precond: P (inverse 0), P^{-1} (1), P^{-T} (2)
  solve     birk_krylov_solve: the linearised two-body system with per-node Jacobians
            ("kepler") or random linear time-invariant systems with constant ones ("lti")
  kkt       birk_kkt_solve on the linearised two-body system
  newton    birk_newton_ivp on the two-body problem, from the circular orbit

Inputs are drawn on the CPU from the seed alone, so that ``exact`` sees the same values.
"""

from __future__ import annotations

import math
import random

import numpy as np
import torch

F64, F32, MIXED, DF32 = 0, 1, 2, 3   # birk_precision
HEADLINE = (1 << 20) + 1


def listed():
    return [
        # one product of a small trajectory: latency of a single call, N not a power of two
        dict(name="product_256_f64", op="product", n_nodes=256, n_x=6, prec=F64, transpose=False),
        # the million-point product of a six-state trajectory
        dict(name="product_1m_f64", op="product", n_nodes=HEADLINE, n_x=6, prec=F64, transpose=False),
        # an adjoint product on a grid whose N is neither a power of two nor smooth
        dict(name="adjoint_100003_f64", op="product", n_nodes=100003, n_x=6, prec=F64, transpose=True),
        # many right-hand sides at once in single precision: 32 x 6 states
        dict(name="product_32rhs_f32", op="product", n_nodes=(1 << 18) + 1, n_x=192, prec=F32, transpose=False),
        # compensated products, eight right-hand sides of six states
        dict(name="product_8rhs_df32", op="product", n_nodes=65537, n_x=48, prec=DF32, transpose=False),
        # a batch of uneven trajectories, as a multi-start search evaluates them
        dict(name="batch64_f64", op="batch", count=64, size_seed=3, log2_lo=8.0, log2_hi=16.0, prec=F64),
        # the preconditioner of a user's own Krylov loop, per-node Jacobians
        dict(name="pinv_1m_f64", op="precond", n_nodes=HEADLINE, n_x=6, prec=F64, inverse=1, per_node=True),
        # a small linear solve, as an inner step of an optimiser runs it: latency
        dict(name="solve_257_f64", op="solve", kind="lti", n_nodes=257, n_x=6, prec=F64, rtol=1e-10),
        # the million-point linear solve
        dict(name="solve_1m_f64", op="solve", kind="kepler", n_nodes=HEADLINE, n_x=6, prec=F64, rtol=1e-10),
        # uneven batch solved in float with double refinement
        dict(name="solve_batch64_mixed", op="solve", kind="lti", count=64, size_seed=3, log2_lo=8.0, log2_hi=16.0,
             prec=MIXED, rtol=1e-11),
        # the saddle-point system of one optimisation step
        dict(name="kkt_65537_f64", op="kkt", n_nodes=65537, n_x=6, prec=F64, rtol=1e-10),
        # a nonlinear trajectory: Newton on the two-body problem over one period
        dict(name="newton_65537_f64", op="newton", n_nodes=65537, n_x=6, prec=F64),
    ]


def _nodes(rng, lo, hi):
    """A node count spread over the logarithm of [lo, hi]: a power of two plus one, or any number."""
    if rng.random() < 0.4:
        p = rng.randint(max(2, math.ceil(math.log2(lo))), math.floor(math.log2(hi - 1)))
        return (1 << p) + 1
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    op = rng.choice(["product", "product", "product", "product", "batch", "bform", "endpoint", "fast_ax", "precond",
                     "precond", "precond", "solve", "solve", "solve", "kkt", "newton"])
    if op in ("product", "bform", "endpoint"):
        nn = _nodes(rng, 16, HEADLINE)
        most = max(1, min(64, 6 * HEADLINE // nn))
        nx = min(most, rng.choice([1, 2, 3, 4, 6, 6, 7, 12, 24, 64]))
        c = dict(op=op, n_nodes=nn, n_x=nx, prec=rng.choice([F64, F64, F64, F32, DF32]))
        if op != "endpoint":
            c["transpose"] = rng.random() < 0.5
        if c["prec"] == DF32 and nn * nx > (1 << 21):
            c["prec"] = F64
        return c
    if op == "batch":
        return dict(op=op, count=rng.randint(2, 64), size_seed=rng.randint(0, 10 ** 6), log2_lo=4.0,
                    log2_hi=round(rng.uniform(8.0, 16.0), 2), prec=rng.choice([F64, F64, F32]))
    if op in ("fast_ax", "precond"):
        nn = _nodes(rng, 16, HEADLINE)
        nx = rng.choice([1, 2, 3, 4, 5, 6, 6, 6, 7, 8, 10, 12])
        while nn * nx * nx > 36 * HEADLINE:
            nx -= 1
        c = dict(op=op, n_nodes=nn, n_x=nx, prec=F64, per_node=rng.random() < 0.7)
        if op == "precond":
            c["inverse"] = rng.choice([0, 1, 1, 2])
            if c["inverse"] != 2 and rng.random() < 0.3:
                c["prec"] = F32
        return c
    if op == "solve":
        prec = rng.choice([F64, F64, MIXED])
        rtol = 1e-10 if prec == F64 else 1e-11
        kind = rng.choice(["kepler", "lti", "batch"])
        if kind == "kepler":
            return dict(op=op, kind=kind, n_nodes=_nodes(rng, 256, HEADLINE), n_x=6, prec=prec, rtol=rtol)
        if kind == "lti":
            return dict(op=op, kind=kind, n_nodes=_nodes(rng, 100, 1 << 17), n_x=rng.choice([1, 2, 4, 6, 6, 8, 12]),
                        prec=prec, rtol=rtol)
        return dict(op=op, kind="lti", count=rng.randint(2, 48), size_seed=rng.randint(0, 10 ** 6), log2_lo=7.0,
                    log2_hi=round(rng.uniform(9.0, 16.0), 2), prec=prec, rtol=rtol)
    if op == "kkt":
        return dict(op=op, n_nodes=_nodes(rng, 256, 1 << 16), n_x=6, prec=F64, rtol=1e-10)
    return dict(op=op, n_nodes=_nodes(rng, 256, 1 << 16), n_x=6, prec=F64)


# ---------------------------------------------------------------- sizes and inputs


def _sizes(case):
    """(node counts, state counts) of the plan's instances."""
    if "count" not in case:
        return [case["n_nodes"]], [case["n_x"]]
    r = random.Random(case["size_seed"])
    nn = [int(round(2.0 ** r.uniform(case["log2_lo"], case["log2_hi"]))) for _ in range(case["count"])]
    nx = [r.choice([4, 6, 12]) for _ in range(case["count"])]
    return nn, nx


def _gen(seed, salt=0):
    g = torch.Generator()
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFFFFFFFFFF)
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, dtype=torch.float64)


def _times(N):
    """tau_j + 1, j = 0..N, as 2 sin^2(j pi / (2 N))."""
    j = torch.arange(N + 1, dtype=torch.float64)
    return 2.0 * torch.sin(j * (math.pi / (2 * N))) ** 2


def _orbit(g, nn):
    """A Keplerian orbit (mu = a = 1, one period, e <= 0.2, random plane): r, v, acceleration
    and time at the nodes, and the circular orbit of the same plane."""
    e = 0.2 * float(torch.rand((), generator=g, dtype=torch.float64))
    q, r = torch.linalg.qr(_randn(g, 3, 3))
    R = q * torch.sign(torch.diagonal(r))
    t = math.pi * _times(nn - 1)

    def at(ec):
        E = t + ec * torch.sin(t)
        for _ in range(8):
            E = E - (E - ec * torch.sin(E) - t) / (1.0 - ec * torch.cos(E))
        c, s = torch.cos(E), torch.sin(E)
        b, d = math.sqrt(1.0 - ec * ec), 1.0 - ec * c
        z = torch.zeros_like(E)
        return R @ torch.stack([c - ec, b * s, z]), R @ torch.stack([-s / d, b * c / d, z])

    pos, vel = at(e)
    p0, v0 = at(0.0)
    acc = -pos / pos.norm(dim=0) ** 3
    return pos, vel, acc, t, torch.cat([p0, v0])


def _kepler(g, nn):
    """Per-node Jacobian (6, 6, N_n) of the linearised two-body problem, and an exact
    solution of it: a combination of the time shift, the rotations and the scaling."""
    pos, vel, acc, t, _ = _orbit(g, nn)
    rn = pos.norm(dim=0)
    rh = pos / rn
    J = torch.zeros(6, 6, nn, dtype=torch.float64)
    for i in range(3):
        J[i, 3 + i] = math.pi
        for k in range(3):
            J[3 + i, k] = math.pi * (3.0 * rh[i] * rh[k] - (1.0 if i == k else 0.0)) / rn ** 3
    c = _randn(g, 5)
    om = c[1:4, None].expand(3, nn)
    chi = torch.cat([c[0] * vel + torch.linalg.cross(om, pos, dim=0) + c[4] * (pos - 1.5 * t * vel),
                     c[0] * acc + torch.linalg.cross(om, vel, dim=0) + c[4] * (-0.5 * vel - 1.5 * t * acc)])
    return J, chi


def _lti(g, nx):
    return _randn(g, nx, nx) / math.sqrt(nx) - 2.0 * torch.eye(nx, dtype=torch.float64), _randn(g, nx)


def _node_jac(g, nn, nx):
    """Smooth per-node Jacobians of any n_x: A0 + A1 sin(5 t) over the interval."""
    a0, _ = _lti(g, nx)
    a1 = _randn(g, nx, nx) / math.sqrt(nx)
    return a0[:, :, None] + a1[:, :, None] * torch.sin(5.0 * _times(nn - 1))


def _inputs(case, seed):
    """The host inputs of a case, by name (double)."""
    g = _gen(seed)
    nn, nx = _sizes(case)
    op = case["op"]
    if op in ("product", "batch", "bform", "endpoint"):
        d = {"v": _randn(g, sum(a * b for a, b in zip(nn, nx)))}
        if op == "endpoint":
            d["xa"] = _randn(g, sum(nx))
        return d
    if op in ("fast_ax", "precond"):
        n, m = nn[0], nx[0]
        if not case["per_node"]:
            J, _ = _lti(g, m)
        else:
            J = _kepler(g, n)[0] if m == 6 else _node_jac(g, n, m)
        return {"J": J, "y": _randn(g, m, n)}
    if op == "solve" and case["kind"] == "kepler":
        J, chi = _kepler(g, nn[0])
        return {"J": J, "chi": chi, "beta": chi[:, :1].expand(6, nn[0]).contiguous()}
    if op == "solve":
        As, xs = zip(*(_lti(g, m) for m in nx))
        return {"A": As, "xa": xs, "J": torch.cat([a.reshape(-1) for a in As]),
                "beta": torch.cat([x[:, None].expand(m, n).reshape(-1) for x, m, n in zip(xs, nx, nn)])}
    if op == "kkt":
        J, chi = _kepler(g, nn[0])
        t = _times(nn[0] - 1)
        c = _randn(g, 6, 3)
        lam = c[:, :1] + c[:, 1:2] * torch.cos(2.0 * t) + c[:, 2:] * torch.sin(3.0 * t)
        h = 1.0 + 0.5 * torch.rand(6, 1, generator=g, dtype=torch.float64) * torch.cos(t)
        Jn, cn, ln = J.numpy(), chi.numpy(), lam.numpy()
        f = h.numpy() * cn + ln - np.einsum("rck,rk->ck", Jn, _ba_t(ln))
        return {"J": J, "h": h, "f": torch.from_numpy(f), "g": chi[:, :1].expand(6, nn[0]).contiguous(),
                "chi": chi, "lam": lam}
    pos, vel, _, _, guess = _orbit(g, nn[0])
    X = torch.cat([pos, vel])
    return {"xa": X[:, 0].contiguous(), "guess": guess, "X": X}


# ---------------------------------------------------------------- prepare and run


def _store(v, prec):
    """A double host vector in the plan's storage type, on the GPU."""
    if prec == F64:
        return v.reshape(-1).cuda()
    if prec == DF32:
        hi = v.reshape(-1).float()
        lo = (v.reshape(-1) - hi.double()).float()
        return torch.stack([hi, lo], dim=1).reshape(-1).cuda()
    return v.reshape(-1).float().cuda()


def prepare(case, seed):
    from paper_2509_01855_amd import birk

    nn, nx = _sizes(case)
    prec = case["prec"]
    d = _inputs(case, seed)
    s = {"case": case, "birk": birk, "plan": birk.birk_plan_create(nn, nx, prec)}
    op = case["op"]
    if op in ("product", "batch", "bform", "endpoint"):
        s["v"] = _store(d["v"], prec)
        s["out"] = torch.empty_like(s["v"])
        if op == "endpoint":
            s["xa"] = d["xa"].cuda()
            s["out"] = torch.empty_like(s["xa"])
    elif op in ("fast_ax", "precond"):
        s["J"] = d["J"].cuda()
        s["y"] = _store(d["y"], F64 if op == "fast_ax" else prec)
        s["out"] = torch.empty_like(s["y"])
        s["kind"] = birk.BIRK_J_PER_NODE if case["per_node"] else birk.BIRK_J_CONSTANT
    elif op == "newton":
        s["xa"], s["guess"] = d["xa"].cuda(), d["guess"].reshape(-1).cuda()
        s["X"] = torch.empty_like(s["guess"])
    else:
        s["J"] = d["J"].cuda()
        s["kind"] = birk.BIRK_J_PER_NODE if s["J"].dim() == 3 else birk.BIRK_J_CONSTANT
        for k in ("beta", "h", "f", "g"):
            if k in d:
                s[k] = d[k].reshape(-1).cuda()
        s["chi"] = torch.empty_like(s["g"] if op == "kkt" else s["beta"])
        if op == "kkt":
            s["lam"] = torch.empty_like(s["chi"])
    return s


def run(s):
    case, birk, plan = s["case"], s["birk"], s["plan"]
    op = case["op"]
    if op in ("product", "batch"):
        (birk.birk_apply_T if case.get("transpose") else birk.birk_apply)(plan, s["v"], s["out"])
        return s["out"]
    if op == "bform":
        (birk.birk_apply_bT if case["transpose"] else birk.birk_apply_b)(plan, s["v"], s["out"])
        return s["out"]
    if op == "endpoint":
        birk.birk_endpoint(plan, s["xa"], s["v"], s["out"])
        return s["out"]
    if op == "fast_ax":
        birk.birk_fast_ax(plan, s["J"], s["y"], s["out"], jac_kind=s["kind"])
        return s["out"]
    if op == "precond":
        birk.birk_precond(plan, s["J"], s["y"], s["out"], case["inverse"], jac_kind=s["kind"])
        return s["out"]
    if op == "solve":
        birk.birk_krylov_solve(plan, s["J"], s["beta"], s["chi"], jac_kind=s["kind"], rtol=case["rtol"])
        return s["chi"]
    if op == "kkt":
        birk.birk_kkt_solve(plan, s["J"], s["g"], s["chi"], lam=s["lam"], h=s["h"], f=s["f"], rtol=case["rtol"])
        return {"chi": s["chi"], "lam": s["lam"]}
    s["X"].copy_(s["guess"])   # the solve overwrites its starting guess
    birk.birk_newton_ivp(plan, s["xa"], s["X"], mu=1.0, scale=math.pi)
    return s["X"]


# ---------------------------------------------------------------- compulsory work


def work(case):
    nn, nx = _sizes(case)
    op, prec = case["op"], case["prec"]
    size = 4 if prec == F32 else 8
    n = sum(a * b for a, b in zip(nn, nx))
    # two real-even transforms (2.5 N log2 N each) and a three-point stencil per component
    product = sum(b * (5.0 * a * math.log2(a) + 10.0 * a) for a, b in zip(nn, nx))
    lu = sum(a * (2.0 / 3.0 * b ** 3 + 4.0 * b * b) for a, b in zip(nn, nx))   # node blocks: factor, solve, apply
    jmul = sum(2.0 * a * b * b for a, b in zip(nn, nx))
    per_node = case.get("per_node", case.get("kind") == "kepler" or op == "kkt")
    jac = 8 * sum(b * b * (a if per_node else 1) for a, b in zip(nn, nx))
    if op in ("product", "batch", "bform"):
        return {"bytes": 2 * n * size, "flops": product}
    if op == "endpoint":
        return {"bytes": n * size + 16 * sum(nx), "flops": 2.0 * n}
    if op == "fast_ax":
        return {"bytes": 16 * n + jac, "flops": product + jmul}
    if op == "precond":
        return {"bytes": 2 * n * size + jac, "flops": lu if case["inverse"] else jmul + 2.0 * n}
    if op == "solve":
        # one preconditioned step and the residual that proves it
        return {"bytes": 16 * n + jac, "flops": lu + 2 * (product + jmul)}
    if op == "kkt":
        # one preconditioned step of the pair and the residual that proves it
        return {"bytes": 5 * 8 * n + jac, "flops": 2 * lu + 4 * (product + jmul)}
    # newton: one step and the residual that proves it
    return {"bytes": 16 * n, "flops": lu + 4 * product}


# ---------------------------------------------------------------- exact values (NumPy, 64 bits)


def _cos_sum(x):
    """sum_j x_j cos(j k pi / N), k = 0..N, along the last axis."""
    N = x.shape[-1] - 1
    y = np.fft.rfft(np.concatenate([x, x[..., -2:0:-1]], axis=-1), axis=-1).real
    k = np.arange(N + 1)
    return 0.5 * (y + x[..., :1] + np.where(k % 2 == 0, 1.0, -1.0) * x[..., -1:])


def _halved(x):
    y = x.copy()
    y[..., 0] *= 0.5
    y[..., -1] *= 0.5
    return y


def _rows(f, x):
    """f over the rows of x, a few at a time."""
    x = np.ascontiguousarray(x)
    return np.concatenate([f(x[i:i + 4]) for i in range(0, x.shape[0], 4)])


def _ba_rows(v):
    """B^a v by its definition on the Chebyshev series: coefficients, term-by-term
    antiderivative (T_{N+1} equals T_{N-1} at the nodes), values; zero at tau = -1."""
    N = v.shape[-1] - 1
    k = np.arange(N + 1)
    sg = np.where(k % 2 == 0, 1.0, -1.0)
    a = sg * (2.0 / N) * _halved(_cos_sum(_halved(v)))
    c = np.zeros_like(a)
    c[..., 1:] = a[..., :-1] / (2.0 * k[1:])
    c[..., 1] += 0.5 * a[..., 0]
    c[..., 1:-1] -= a[..., 2:] / (2.0 * k[1:-1])
    c[..., N - 1] += a[..., N] / (2.0 * (N + 1))
    c *= sg
    c[..., 0] = -c[..., 1:].sum(axis=-1)
    return _cos_sum(c)


def _ba_t_rows(g):
    N = g.shape[-1] - 1
    k = np.arange(N + 1)
    sg = np.where(k % 2 == 0, 1.0, -1.0)
    p = _cos_sum(g)
    q = sg * (p - p[..., :1])
    q[..., 0] = 0.0
    a = np.zeros_like(q)
    a[..., :-1] = q[..., 1:] / (2.0 * k[1:])
    a[..., 0] += 0.5 * q[..., 1]
    a[..., 2:] -= q[..., 1:-1] / (2.0 * k[1:-1])
    a[..., N] += q[..., N - 1] / (2.0 * (N + 1))
    return _halved(_cos_sum(_halved(sg * a))) * (2.0 / N)


def _ba(v):
    return _rows(_ba_rows, v)


def _ba_t(g):
    return _rows(_ba_t_rows, g)


def _cc(N):
    """Clenshaw-Curtis weights."""
    k = np.arange(N + 1, dtype=np.float64)
    m = np.where(k % 2 == 0, 2.0 / (1.0 - np.where(k == 1, 0.0, k) ** 2), 0.0)
    return (2.0 / N) * _halved(_cos_sum(_halved(m)))


def _affine_states(A, b):
    """S_0 = 0, S_{k+1} = A_k S_k + b_k: the states S_k before each node.  Chunks of about
    sqrt(n) nodes side by side, then from chunk to chunk, then the chunks again."""
    n, m = b.shape
    L = max(1, int(math.sqrt(n)))
    C = -(-n // L)
    Ap = np.broadcast_to(np.eye(m), (C * L, m, m)).copy()
    bp = np.zeros((C * L, m))
    Ap[:n], bp[:n] = A, b
    Ap, bp = Ap.reshape(C, L, m, m), bp.reshape(C, L, m)
    M = np.broadcast_to(np.eye(m), (C, m, m)).copy()
    c = np.zeros((C, m))
    for j in range(L):
        M = Ap[:, j] @ M
        c = (Ap[:, j] @ c[:, :, None])[:, :, 0] + bp[:, j]
    S = np.zeros((C, m))
    for i in range(C - 1):
        S[i + 1] = M[i] @ S[i] + c[i]
    out = np.zeros((C, L, m))
    for j in range(L):
        out[:, j] = S
        S = (Ap[:, j] @ S[:, :, None])[:, :, 0] + bp[:, j]
    return out.reshape(C * L, m)[:n]


def _precond(J, y, inverse):
    m, n = y.shape
    w = _cc(n - 1)
    Jn = J if J.ndim == 3 else np.broadcast_to(J[:, :, None], (m, m, n))
    if inverse == 0:
        u = w * np.einsum("rck,ck->rk", Jn, y)
        return y - (np.cumsum(u, axis=1) - 0.5 * u)
    W = np.ascontiguousarray(np.moveaxis(Jn, 2, 0)) * w[:, None, None]
    yk = np.ascontiguousarray(y.T)
    if inverse == 2:
        W, yk = np.ascontiguousarray(np.swapaxes(W, 1, 2)[::-1]), yk[::-1]
    Ki = np.linalg.inv(np.eye(m) - 0.5 * W)
    if inverse == 1:
        # S <- S + W K^{-1} (y + S), xi = K^{-1} (y + S)
        H = W @ Ki
        S = _affine_states(np.eye(m) + H, (H @ yk[:, :, None])[:, :, 0])
        return (Ki @ (yk + S)[:, :, None])[:, :, 0].T
    # T <- T + x, x = K^{-1} (y + W T)
    T = _affine_states(np.eye(m) + Ki @ W, (Ki @ yk[:, :, None])[:, :, 0])
    x = (Ki @ (yk + (W @ T[:, :, None])[:, :, 0])[:, :, None])[:, :, 0]
    return x[::-1].T


def _parts(v, nn, nx):
    off = 0
    for a, b in zip(nn, nx):
        yield v[off:off + a * b].reshape(b, a)
        off += a * b


def _laid_out(x, prec):
    """An exact double result in the plan's storage layout."""
    x = np.ascontiguousarray(x).reshape(-1)
    if prec != DF32:
        return x
    hi = x.astype(np.float32).astype(np.float64)
    return np.stack([hi, x - hi], axis=1).reshape(-1)


def exact(case, seed):
    nn, nx = _sizes(case)
    op, prec = case["op"], case["prec"]
    d = _inputs(case, seed)

    def stored(t):
        t = t.float().double() if prec in (F32, MIXED) else t
        return t.numpy()

    if op in ("product", "batch", "bform"):
        v = stored(d["v"])
        outs = []
        for x in _parts(v, nn, nx):
            if case.get("transpose"):
                o = _ba_t(x)
                if op == "bform":
                    o = o - _cc(x.shape[1] - 1) * x.sum(axis=1, keepdims=True)
            else:
                o = _ba(x)
                if op == "bform":
                    o = o - o[:, -1:]
            outs.append(o.reshape(-1))
        return _laid_out(np.concatenate(outs), prec)
    if op == "endpoint":
        x = stored(d["v"]).reshape(nx[0], nn[0])
        return d["xa"].numpy() + x @ _cc(nn[0] - 1)
    if op == "fast_ax":
        J, x = d["J"].numpy(), d["y"].numpy()
        return (x - _ba(np.einsum("rck,ck->rk" if J.ndim == 3 else "rc,ck->rk", J, x))).reshape(-1)
    if op == "precond":
        if nn[0] * nx[0] ** 2 > (1 << 26):
            return None
        return np.ascontiguousarray(_precond(d["J"].numpy(), stored(d["y"]), case["inverse"])).reshape(-1)
    if op == "solve" and case["kind"] == "kepler":
        return d["chi"].numpy().reshape(-1)
    if op == "solve":
        outs = []
        for A, xa, n in zip(d["A"], d["xa"], nn):
            E = torch.linalg.matrix_exp(_times(n - 1)[:, None, None] * A)
            outs.append((E @ xa).T.reshape(-1))
        return torch.cat(outs).numpy()
    if op == "kkt":
        return {"chi": d["chi"].numpy().reshape(-1), "lam": d["lam"].numpy().reshape(-1)}
    return d["X"].numpy().reshape(-1)
