"""P^{-1} and P^{-T} with one J per instance on long plans of n_x = 2 to 5, where a lane carries
four nodes, at the edges of its rule and tiles: 10^5 nodes and one less, whole rounds of 256 and
one more node, two rounds a tile (2^19 + 1), uneven batches with one-launch instances among them;
n_x = 1 and 6 beside them keep their kernels.  Against the same J given per node, whose kernels
the scan tests hold to the oracle: 1e-12 of the largest value (2e-6 where a float plan stores the
result), and one size against the oracle itself.  The solves use J xi from the same pass."""

import numpy as np
import pytest

from oracle import birkhoff as bk
from oracle import system as sy
from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dev, host, rel_err

pytestmark = pytest.mark.gpu

PLANS = {"below": [99999], "at": [100000], "rounds": [131072], "one more": [131073], "two rounds": [524289],
         "batch": [3, 400, 512, 513, 769, 20000, 30001, 49999], "many": [2000] * 60 + [500] * 5}


def _jacobians(Nns, nx, seed):
    As = [wl.lti_matrix(np.random.default_rng([101, seed, i]), nx) for i in range(len(Nns))]
    const = np.concatenate([A.ravel() for A in As])
    per = np.concatenate([np.repeat(A.ravel(), n) for A, n in zip(As, Nns)])   # entry (r, c) contiguous over nodes
    return As, const, per


@pytest.mark.parametrize("nx", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("plan", list(PLANS))
def test_inverse_and_transpose(plan, nx):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    Nns = PLANS[plan]
    announce(f"four nodes a lane: {plan} n_x={nx}")
    As, const, per = _jacobians(Nns, nx, nx)
    y = wl.random_vectors([102, nx], (nx * sum(Nns),))[0]
    Jc, Jp = dev(const, torch.float64), dev(per, torch.float64)
    for prec, modes in ((B.BIRK_F64, (1, 2)), (B.BIRK_F32, (1,))):
        p = B.birk_plan_create(Nns, [nx] * len(Nns), prec)
        v = dev(y, torch.float64 if prec == B.BIRK_F64 else torch.float32)
        for inv in modes:
            a, b = torch.full_like(v, float("nan")), torch.full_like(v, float("nan"))
            B.birk_precond(p, Jc, v, a, inv, B.BIRK_J_CONSTANT)
            B.birk_precond(p, Jp, v, b, inv, B.BIRK_J_PER_NODE)
            torch.cuda.synchronize()
            assert rel_err(host(a), host(b)) <= (1e-12 if prec == B.BIRK_F64 else 2e-6), (prec, inv)
            if plan == "at" and prec == B.BIRK_F64 and inv == 1 and nx == 3:
                ref = sy.precond_inverse(bk.weights(Nns[0] - 1) if Nns[0] < 5000 else B.birk_weights(p), As[0], y)
                assert rel_err(host(a), ref) <= 1e-12
        p.destroy()


@pytest.mark.parametrize("nx", [2, 5])
@pytest.mark.parametrize("prec", ["f64", "mixed"])
def test_solve_and_singular_pivot(nx, prec):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    Nn = 131073
    announce(f"four nodes a lane: solves n_x={nx} {prec}")
    As, const, per = _jacobians([Nn], nx, 7)
    b = dev(sy.beta_vector(np.arange(1.0, nx + 1.0), Nn), torch.float64)
    xs = []
    p = B.birk_plan_create([Nn], [nx], B.BIRK_F64 if prec == "f64" else B.BIRK_F32_REFINE_F64)
    for J, kind in ((const, B.BIRK_J_CONSTANT), (per, B.BIRK_J_PER_NODE)):
        x = torch.full_like(b, float("nan"))
        B.birk_krylov_solve(p, dev(J, torch.float64), b, x, kind, rtol=1e-13 if prec == "f64" else 1e-11)
        xs.append(host(x))
    # both to their residual, with condition numbers below 100
    assert rel_err(xs[0], xs[1]) <= (1e-11 if prec == "f64" else 1e-9)
    w = B.birk_weights(p)
    bad = (2.0 / w[Nn // 3]) * np.eye(nx)
    x = torch.full_like(b, float("nan"))
    info = B.birk_krylov_solve(p, dev(bad.ravel(), torch.float64), b, x, B.BIRK_J_CONSTANT, raise_on_error=False)
    p.destroy()
    assert info["status"] == B.BIRK_ERR_SINGULAR
