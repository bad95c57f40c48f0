"""Tuning a plan whose lengths share a class of the chirp tuner but not its splits: lengths of
3 2^m, 2^m, 5 2^m and 3 2^(m+1) side by side, the shortest of which allow fewer splits than the
longest.  The tuned products against the untuned ones: 1e-13 (double) and 2e-6 (float) of the
largest value, as in the other tuner tests (rounding order only)."""

import numpy as np
import pytest

from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dev, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 2e-6), ("mixed", 2e-6)])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_mixed_lengths_of_a_class(prec, tol, shift):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    Nns = [(n << shift) + 1 for n in (1404, 1532, 1790, 2019, 2300, 2559, 2600, 2729)]
    nx = [1, 2, 3, 1, 2, 1, 3, 2]
    announce(f"tuned class of mixed lengths {Nns} {prec}")
    x = wl.random_vectors([73, shift], (sum(a * b for a, b in zip(Nns, nx)),))[0]
    plan = B.birk_plan_create(Nns, nx, {"f64": B.BIRK_F64, "f32": B.BIRK_F32, "mixed": B.BIRK_F32_REFINE_F64}[prec])
    v = dev(x, torch.float64 if prec == "f64" else torch.float32)

    def both():
        outs = []
        for f in (B.birk_apply, B.birk_apply_T):
            out = torch.full_like(v, float("nan"))
            f(plan, v, out)
            torch.cuda.synchronize()
            outs.append(host(out).astype(np.float64))
        return outs

    before = both()
    B.birk_plan_tune(plan)
    after = both()
    B.birk_plan_tune(plan)
    again = both()
    plan.destroy()
    o = 0
    for n, m in zip(Nns, nx):
        for a, b, c in zip(before, after, again):
            assert rel_err(b[o:o + n * m], a[o:o + n * m]) <= tol, n
            assert rel_err(c[o:o + n * m], a[o:o + n * m]) <= tol, n
        o += n * m
