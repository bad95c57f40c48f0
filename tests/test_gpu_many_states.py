"""J x and J^T x for any n_x: the entry points that take plans with n_x > 12 (FastAX, GMRES and
MINRES without the preconditioner) on one plan whose instances have 4, 12, 13 and 20 states.
References: the oracle's dense operators and solutions.  Bars: FastAX 1e-12 of the largest value;
the solves run to rtol 1e-13 and the systems have condition numbers below 100 (constant,
dissipative A), so 1e-11."""

import numpy as np
import pytest

from oracle import kkt
from oracle import system as sy
from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dense_Ba, dev, host, rel_err

pytestmark = pytest.mark.gpu

NN, NX = [40, 65, 33, 51], [4, 13, 20, 12]


def _instances(per_node):
    out = []
    for k, (Nn, nx) in enumerate(zip(NN, NX)):
        rng = np.random.default_rng([91, k])
        A = wl.lti_matrix(rng, nx)
        if per_node:
            t = np.linspace(0.0, 1.0, Nn)
            A = A[:, :, None] + 0.3 / np.sqrt(nx) * rng.standard_normal((nx, nx))[:, :, None] * np.cos(3.0 * t)
        out.append((Nn, nx, A))
    return out


def _plan(B, prec, insts):
    import torch
    plan = B.birk_plan_create(NN, NX, prec)
    J = dev(np.concatenate([A.ravel() for _, _, A in insts]), torch.float64)
    jk = B.BIRK_J_PER_NODE if insts[0][2].ndim == 3 else B.BIRK_J_CONSTANT
    return plan, J, jk


@pytest.mark.parametrize("per_node", [0, 1])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_fast_ax(per_node, prec):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    announce(f"FastAX n_x {NX} per_node={per_node} {prec}")
    insts = _instances(per_node)
    plan, J, jk = _plan(B, B.BIRK_F64 if prec == "f64" else B.BIRK_F32, insts)
    x = wl.random_vectors([92, 0], (plan.length,))[0]
    out = torch.full((plan.length,), float("nan"), dtype=torch.float64, device="cuda")
    B.birk_fast_ax(plan, J, dev(x, torch.float64), out, jac_kind=jk)
    torch.cuda.synchronize()
    plan.destroy()
    got, o = host(out), 0
    for Nn, nx, A in insts:
        ref = sy.dense_A(Nn - 1, A, dense_Ba(Nn - 1)) @ x[o:o + Nn * nx]
        assert rel_err(got[o:o + Nn * nx], ref) <= 1e-12, nx
        o += Nn * nx


@pytest.mark.parametrize("per_node", [0, 1])
@pytest.mark.parametrize("method", ["gmres", "gmres_mixed", "minres"])
def test_solves_without_preconditioner(per_node, method):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    announce(f"{method} without preconditioner n_x {NX} per_node={per_node}")
    insts = _instances(per_node)
    mixed = method == "gmres_mixed"
    plan, J, jk = _plan(B, B.BIRK_F32_REFINE_F64 if mixed else B.BIRK_F64, insts)
    xa = [np.random.default_rng([93, k]).standard_normal(nx) for k, nx in enumerate(NX)]
    beta = np.concatenate([sy.beta_vector(a, Nn) for a, Nn in zip(xa, NN)])
    b = dev(beta, torch.float64)
    chi, lam = torch.full_like(b, float("nan")), torch.full_like(b, float("nan"))
    if method == "minres":
        B.birk_kkt_solve(plan, J, b, chi, lam=lam, jac_kind=jk, rtol=1e-13, use_precond=0, max_iter=2000)
    else:
        B.birk_krylov_solve(plan, J, b, chi, jk, rtol=1e-11 if mixed else 1e-13, use_precond=0)
    torch.cuda.synchronize()
    plan.destroy()
    got, gl, o = host(chi), host(lam), 0
    for Nn, nx, A in insts:
        n = Nn * nx
        D = sy.dense_A(Nn - 1, A, dense_Ba(Nn - 1))
        ref = sy.solve_dense(D, beta[o:o + n])
        assert rel_err(got[o:o + n], ref) <= (1e-9 if mixed else 1e-11), nx
        if method == "minres":
            _, rl = kkt.kkt_solve_dense(kkt.dense_K(Nn - 1, A, np.ones(n), dense_Ba(Nn - 1)), np.zeros(n),
                                        beta[o:o + n])
            assert rel_err(gl[o:o + n], rl) <= 1e-11, nx
        o += n
