"""GPU parity of the scans behind P^{-1} and P^{-T} at the sizes where their split
changes: around one chunk (16 nodes) and one wave (64), the last instance that one workgroup
holds and the first that it does not, one and two groups of tiles, one and two rounds per
tile; forward and transposed, one J and J per node, double and float; alone and side by side
in one plan, whose launches then hold all kinds, bit for bit.  Reference: block substitution in
NumPy.  Bars as in the preconditioner tests: 1e-12 (double), 2e-6 (float storage) of the
largest value, times 1 + N / 1e5 for the growth of the chain's rounding."""

import numpy as np
import pytest

from oracle import birkhoff as bk
from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dev, host, rel_err

pytestmark = pytest.mark.gpu

WAVES = {1: 16, 2: 16, 3: 12, 4: 12, 5: 8, 6: 7, 7: 5, 8: 4}   # tiles per CU in one round


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk
    return birk


def _jac(nx, Nn, per_node, seed):
    rng = np.random.default_rng([seed, nx, Nn])
    A0 = rng.standard_normal((nx, nx)) / np.sqrt(nx) - 2.0 * np.eye(nx)
    if not per_node:
        return A0
    A1 = rng.standard_normal((nx, nx)) / np.sqrt(nx)
    return A0[:, :, None] + A1[:, :, None] * np.sin(5.0 * np.linspace(-1.0, 1.0, Nn))


def _substitute(J, w, y, back):
    """P^{-1} y, or P^{-T} y (back): y[n_x, Nn], J[n_x, n_x] or [n_x, n_x, Nn]."""
    nx, Nn = y.shape
    Jn = np.broadcast_to(J[:, :, None], (nx, nx, Nn)) if J.ndim == 2 else J
    Jn = np.ascontiguousarray(np.moveaxis(Jn, 2, 0))
    K = np.eye(nx) - 0.5 * w[:, None, None] * Jn
    H = np.linalg.solve(K, w[:, None, None] * Jn)
    S = np.zeros(nx)
    out = np.empty_like(y)
    for k in (range(Nn - 1, -1, -1) if back else range(Nn)):
        if back:
            x = y[:, k] + H[k].T @ (S + 0.5 * y[:, k])
            S = S + x
            out[:, k] = x
        else:
            u = y[:, k] + S
            v = H[k] @ u
            out[:, k] = u + 0.5 * v
            S = S + v
    return out


def _run(B, parts, prec, inverse, per_node, J, y):
    import torch
    plan = B.birk_plan_create([n for n, _ in parts], [m for _, m in parts], B.BIRK_F64 if prec == "f64" else B.BIRK_F32)
    v = dev(y, torch.float64 if prec == "f64" else torch.float32)
    out = torch.full_like(v, float("nan"))
    B.birk_precond(plan, dev(J, torch.float64), v, out, inverse, B.BIRK_J_PER_NODE if per_node else B.BIRK_J_CONSTANT)
    torch.cuda.synchronize()
    r = host(out)
    plan.destroy()
    return r


def _check(B, parts, inverse, prec, per_node):
    announce(f"scan {parts} inverse={inverse} {prec} per_node={per_node}")
    Js = [_jac(m, n, per_node, 3) for n, m in parts]
    ys = [np.random.default_rng([9, n, m]).standard_normal((m, n)) for n, m in parts]
    if prec == "f32":
        ys = [y.astype(np.float32).astype(np.float64) for y in ys]
    flat = lambda a: np.concatenate([x.ravel() for x in a])
    mixed = _run(B, parts, prec, inverse, per_node, flat(Js), flat(ys))
    o = 0
    for (n, m), J, y in zip(parts, Js, ys):
        got = mixed[o:o + m * n]
        o += m * n
        ref = _substitute(J, bk.weights(n - 1), y, inverse == 2)
        bar = (1e-12 if prec == "f64" else 2e-6) * (1.0 + n / 1e5)
        assert rel_err(got.reshape(m, n).astype(np.float64), ref) <= bar, (n, m)
        if len(parts) > 1:
            assert np.array_equal(_run(B, [(n, m)], prec, inverse, per_node, J.ravel(), y.ravel()), got), (n, m)


@pytest.mark.parametrize("per_node", [False, True])
@pytest.mark.parametrize("inverse,prec", [(1, "f64"), (1, "f32"), (2, "f64")])
@pytest.mark.parametrize("nx", range(1, 9))
def test_split_edges(B, nx, inverse, prec, per_node):
    # 64 nodes a wave; 8, 7, 5, 4 waves a workgroup at n_x <= 5, 6, 7, 8; 64 tiles a group
    most = 64 * {6: 7, 7: 5, 8: 4}.get(nx, 8)
    _check(B, [(n, nx) for n in (3, 16, 17, 63, 64, 65, most, most + 1, 4096, 4097, 4161)], inverse, prec, per_node)


@pytest.mark.parametrize("inverse", [1, 2])
@pytest.mark.parametrize("nx", [2, 4, 6, 8])
def test_rounds(B, nx, inverse):
    n = 64 * 256 * WAVES[nx]   # one round per tile up to here, two from the next node on
    for nn in (n, n + 1):
        _check(B, [(nn, nx)], inverse, "f64", nx == 6)


@pytest.mark.parametrize("per_node", [False, True])
@pytest.mark.parametrize("inverse,prec", [(1, "f64"), (1, "f32"), (2, "f64")])
@pytest.mark.parametrize("nx", range(9, 13))
def test_split_edges_wide(B, nx, inverse, prec, per_node):
    # sixteen nodes a tile (two rounds from 16385 nodes), 32 tiles a group
    sizes = (3, 15, 16, 17, 32, 33, 512, 513, 528, 529, 1025) + ((16384, 16385) if nx == 12 else ())
    _check(B, [(n, nx) for n in sizes], inverse, prec, per_node)
