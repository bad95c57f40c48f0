"""GMRES where its vector passes change shape: plans whose instances are one tile of 2048
elements each (one launch per step orthogonalises) against the same instances beside a longer
one (several launches), bit for bit; and against the dense oracle, 1e-9 relative for a residual
of 1e-11 (condition numbers below 100).  Steps: 1 to past 8
basis vectors (no preconditioner), so that every bound on their number is met; x0 given and
not."""

import numpy as np
import pytest

from oracle import system as sy
from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dense_Ba, dev, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk
    return birk


def _solve(B, insts, x0, use_precond, mixed):
    import torch
    plan = B.birk_plan_create([i.N_n for i in insts], [i.n_x for i in insts],
                              B.BIRK_F32_REFINE_F64 if mixed else B.BIRK_F64)
    J = dev(np.concatenate([i.J.ravel() for i in insts]), torch.float64)
    beta = dev(np.concatenate([sy.beta_vector(np.arange(1.0, i.n_x + 1.0), i.N_n) for i in insts]), torch.float64)
    chi = torch.full_like(beta, float("nan")) if x0 is None else dev(np.concatenate(x0), torch.float64)
    B.birk_krylov_solve(plan, J, beta, chi, B.BIRK_J_CONSTANT, rtol=1e-11, use_x0=0 if x0 is None else 1,
                        use_precond=use_precond)
    torch.cuda.synchronize()
    plan.destroy()
    out, o = [], 0
    for i in insts:
        out.append(host(chi)[o:o + i.N_n * i.n_x])
        o += i.N_n * i.n_x
    return out


@pytest.mark.parametrize("use_precond,mixed", [(0, False), (1, False), (1, True)])
@pytest.mark.parametrize("with_x0", [False, True])
def test_one_tile_and_more(B, use_precond, mixed, with_x0):
    announce(f"one-tile solves precond={use_precond} mixed={mixed} x0={with_x0}")
    # 16, 341 * 6 = 2046 and 512 * 4 = 2048 elements (one tile); 513 * 4 = 2052 (two)
    small = [wl.lti_instance(3, 8, 2), wl.lti_instance(4, 341, 6), wl.lti_instance(5, 512, 4)]
    big = wl.lti_instance(6, 513, 4)
    rng = np.random.default_rng(5)
    x0 = [rng.standard_normal(i.N_n * i.n_x) for i in small + [big]] if with_x0 else None
    alone = _solve(B, small, x0[:3] if with_x0 else None, use_precond, mixed)
    mixed_plan = _solve(B, small + [big], x0, use_precond, mixed)
    for k, i in enumerate(small + [big]):
        A = sy.dense_A(i.N_n - 1, i.J, dense_Ba(i.N_n - 1))
        ref = sy.solve_dense(A, sy.beta_vector(np.arange(1.0, i.n_x + 1.0), i.N_n))
        assert rel_err(mixed_plan[k], ref) <= 1e-9
    # each instance alone: the small ones by the one launch, the long one by the several
    for k, i in enumerate(small + [big]):
        one = _solve(B, [i], [x0[k]] if with_x0 else None, use_precond, mixed)[0]
        assert np.array_equal(one, mixed_plan[k]), k
        if k < 3:
            assert np.array_equal(one, alone[k]), k
