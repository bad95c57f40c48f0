"""Every two-step split of the chirp convolutions that the tuner may choose, whether or not it
would: BIRK_BLU_SPLIT sets the nominal M1 = 2^x of the lengths that allow it, x = 7..12, for
lengths just under 3, 4, 5 and 6 times a power of two in classes up to 2^20, so that every column
transform (R 2^A) and row transform of the kernels runs.  Against the products with the default
splits, whose oracle parity the length tests hold: rounding order only, 1e-13 (double and
double-float) and 2e-6 (float) of the largest value, as in the tuner tests."""

import numpy as np
import pytest

from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dev, from_df32, host, rel_err, to_df32

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 2e-6, "df32": 1e-13}


@pytest.mark.parametrize("prec", ["f64", "f32", "df32"])
@pytest.mark.parametrize("base", [3, 4, 5, 6])
def test_products_at_every_split(monkeypatch, base, prec):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    Nns = [n for n in ((base << k) // 4 for k in range(11, 18)) if n > 1400]
    x = wl.random_vectors([74, base], (sum(Nns),))[0]
    v = dev(to_df32(x[None, :])[0]) if prec == "df32" else dev(x, torch.float64 if prec == "f64" else torch.float32)

    def both():
        plan = B.birk_plan_create(Nns, [1] * len(Nns), {"f64": B.BIRK_F64, "f32": B.BIRK_F32, "df32": B.BIRK_DF32}[prec])
        outs = []
        for f in (B.birk_apply, B.birk_apply_T):
            out = torch.full_like(v, float("nan"))
            f(plan, v, out)
            torch.cuda.synchronize()
            r = host(out)
            outs.append(from_df32(r[None, :])[0] if prec == "df32" else r.astype(np.float64))
        plan.destroy()
        return outs

    monkeypatch.delenv("BIRK_BLU_SPLIT", raising=False)
    default = both()
    for split in range(7, 13):
        announce(f"chirp split M1 = 2^{split} N_n {Nns} {prec}")
        monkeypatch.setenv("BIRK_BLU_SPLIT", str(split))
        o = 0
        got = both()
        for n in Nns:
            for a, b in zip(got, default):
                assert rel_err(a[o:o + n], b[o:o + n]) <= TOL[prec], (split, n)
            o += n
