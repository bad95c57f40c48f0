"""birk_krylov_solve returns with its stream idle and chi in place, also where no cycle of the
solve writes chi: a zero right-hand side, a non-finite one, a singular pivot.  chi (400 MB, so
that clearing it takes some 100 us) is full of NaN before the call; right after it the plan's
stream has nothing left to do, and a read of chi on another stream finds zeros."""

import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "mixed"])
def test_chi_is_there_on_return(prec):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    Nn, nx = (1 << 23) + 1, 6
    st, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(st):
        plan = B.birk_plan_create([Nn], [nx], B.BIRK_F64 if prec == "f64" else B.BIRK_F32_REFINE_F64, stream=st)
    w = B.birk_weights(plan)
    eye = np.eye(nx)
    small, singular = -2.0 * eye, (2.0 / w[Nn // 2]) * eye
    cases = [("zero", small, 0.0, B.BIRK_OK), ("non-finite", small, float("inf"), B.BIRK_ERR_NONFINITE),
             ("singular", singular, 1.0, B.BIRK_ERR_SINGULAR)]
    chi = torch.empty(nx * Nn, dtype=torch.float64, device="cuda")
    for name, J, b, want in cases:
        announce(f"solve returns with chi, {prec}, {name} right-hand side or pivot")
        Jd = torch.from_numpy(J.ravel().copy()).to("cuda")
        beta = torch.full_like(chi, b)
        chi.fill_(float("nan"))
        torch.cuda.synchronize()
        info = B.birk_krylov_solve(plan, Jd, beta, chi, B.BIRK_J_CONSTANT, raise_on_error=False, restart=1)
        idle = st.query()
        with torch.cuda.stream(other):
            copy = chi.clone()
        torch.cuda.synchronize()
        assert info["status"] == want, (name, info)
        assert idle, name
        assert not bool(torch.any(copy != 0.0)), name   # NaN != 0 too
    plan.destroy()
