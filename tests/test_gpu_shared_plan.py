"""One plan through both solvers: MINRES on the KKT form first, then GMRES, whose reduction
scratch the first must not have set up in a size of its own.  Both solve A chi = beta to
1e-12; they agree with a GMRES solve on a fresh plan to 1e-10 (the system's condition number
is below 100)."""

import numpy as np
import pytest

from oracle import system as sy
from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dev, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Nn", [257, 4097])
def test_kkt_then_gmres(Nn):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    announce(f"KKT then GMRES on one plan Nn={Nn}")
    inst = wl.lti_instance(4, Nn)
    J = dev(inst.J.ravel(), torch.float64)
    beta = dev(sy.beta_vector(np.arange(1.0, inst.n_x + 1.0), Nn), torch.float64)
    chi = [torch.zeros_like(beta) for _ in range(3)]
    plan = B.birk_plan_create([Nn], [inst.n_x], B.BIRK_F64)
    B.birk_kkt_solve(plan, J, beta, chi[0], jac_kind=B.BIRK_J_CONSTANT, rtol=1e-12)
    B.birk_krylov_solve(plan, J, beta, chi[1], B.BIRK_J_CONSTANT, rtol=1e-12)
    plan.destroy()
    fresh = B.birk_plan_create([Nn], [inst.n_x], B.BIRK_F64)
    B.birk_krylov_solve(fresh, J, beta, chi[2], B.BIRK_J_CONSTANT, rtol=1e-12)
    torch.cuda.synchronize()
    fresh.destroy()
    assert np.array_equal(host(chi[1]), host(chi[2]))
    assert rel_err(host(chi[0]), host(chi[2])) <= 1e-10
