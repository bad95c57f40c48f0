"""Each component of a product keeps its own accuracy and its own non-finite values where a
power-of-two N >= 512 is concerned (shorter ones and the chirp lengths transform two components
as one complex vector).  Components of one instance 10^3 and 10^6 times apart, each judged
against its own largest value with the bars of the product tests (1e-12, 2e-5, 1e-13; oracle in
extended precision); and an infinity or NaN in one component, which must leave the bits of all
others as they are."""

import numpy as np
import pytest

from oracle import birkhoff as bk
from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dev, from_df32, host, rel_err, to_df32

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 2e-5, "df32": 1e-13}
SIZES = [513, 1025, 2049, 4097]   # whole products in LDS up to 2049, three passes from there on


def _products(Nn, nx, prec, xs, transpose):
    import torch
    from paper_2509_01855_amd import birk as B
    plan = B.birk_plan_create(Nn, nx, {"f64": B.BIRK_F64, "f32": B.BIRK_F32, "df32": B.BIRK_DF32}[prec])
    outs = []
    for x in xs:
        v = dev(to_df32(x[None, :])[0]) if prec == "df32" else dev(x, torch.float64 if prec == "f64" else torch.float32)
        out = torch.full_like(v, float("nan"))
        (B.birk_apply_T if transpose else B.birk_apply)(plan, v, out)
        torch.cuda.synchronize()
        r = host(out)
        outs.append(from_df32(r[None, :])[0] if prec == "df32" else r.astype(np.float64))
    plan.destroy()
    return outs


@pytest.mark.parametrize("prec", ["f64", "f32", "df32"])
@pytest.mark.parametrize("transpose", [0, 1])
@pytest.mark.parametrize("ratio", [1e3, 1e6])
def test_components_far_apart(prec, transpose, ratio):
    announce(f"component ratio {ratio:g} {prec} transpose={transpose}")
    nx = [2, 6, 3, 2]
    xs = []
    for n, m in zip(SIZES, nx):
        x = wl.random_vectors([81, n], (m, n))[0]
        x[::2] *= ratio
        if prec == "f32":
            x = x.astype(np.float32).astype(np.float64)   # what the product is given
        xs.append(x)
    out = _products(SIZES, nx, prec, [np.concatenate([x.ravel() for x in xs])], transpose)[0]
    o = 0
    for n, m, x in zip(SIZES, nx, xs):
        part = out[o:o + m * n].reshape(m, n)
        o += m * n
        ref = bk.apply_Ba_extended(n - 1, x, transpose=bool(transpose))
        for r in range(m):
            assert rel_err(part[r], ref[r]) <= TOL[prec], (n, r)


@pytest.mark.parametrize("prec", ["f64", "f32", "df32"])
@pytest.mark.parametrize("transpose", [0, 1])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_non_finite_component_stays_alone(prec, transpose, bad):
    announce(f"non-finite component {bad} {prec} transpose={transpose}")
    nx = [2, 6, 3, 2]
    xs = [wl.random_vectors([82, n], (m, n))[0] for n, m in zip(SIZES, nx)]
    hit = [x.copy() for x in xs]
    for x in hit:
        x[0, 7] = bad
    clean, got = _products(SIZES, nx, prec, [np.concatenate([x.ravel() for x in s]) for s in (xs, hit)], transpose)
    o = 0
    for n, m in zip(SIZES, nx):
        a, b = clean[o:o + m * n].reshape(m, n), got[o:o + m * n].reshape(m, n)
        o += m * n
        assert not np.isfinite(b[0]).any()
        assert np.array_equal(a[1:], b[1:]), n
