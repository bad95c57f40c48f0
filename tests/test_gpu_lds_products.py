"""GPU parity of the one-launch products (N <= 2048 a power of two, or any N with
3N <= 4096) at the sizes where the kernel changes: the shortest grids, transform lengths
below and above one wave's 512 points, both sides of the last Bluestein length and of the
last power of two, and one plan that mixes them all, so that workgroups hold one, several
and a partial set of pairs.  Reference: the oracle's extended-precision product; bars as in
the product tests (1e-12, 2e-5, 1e-13 relative to the largest value)."""

import numpy as np
import pytest

from oracle import birkhoff as bk
from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dev, from_df32, host, rel_err, to_df32

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 2e-5, "df32": 1e-13}
#      N = 2, 3, 4 | M = 16, 64 | L = 64 | M = 512, 1024 | L = 512, 1024 | last M = 4096, first beyond | L = 4096, beyond
EDGES = [3, 4, 5, 6, 22, 33, 171, 172, 257, 513, 1366, 1367, 2049, 2050]


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk
    return birk


def _run(B, Nn, nx, prec, x, transpose):
    import torch
    plan = B.birk_plan_create(Nn, nx, {"f64": B.BIRK_F64, "f32": B.BIRK_F32, "df32": B.BIRK_DF32}[prec])
    if prec == "df32":
        v = dev(to_df32(x[None, :])[0])
    else:
        v = dev(x, torch.float64 if prec == "f64" else torch.float32)
    out = torch.full_like(v, float("nan"))
    (B.birk_apply_T if transpose else B.birk_apply)(plan, v, out)
    torch.cuda.synchronize()
    r = host(out)
    plan.destroy()
    return from_df32(r[None, :])[0] if prec == "df32" else r.astype(np.float64)


@pytest.mark.parametrize("prec", ["f64", "f32", "df32"])
@pytest.mark.parametrize("transpose", [0, 1])
def test_edges_alone_and_mixed(B, prec, transpose):
    announce(f"one-launch products {prec} transpose={transpose}")
    nx = [1 + (3 * i) % 5 for i in range(len(EDGES))]    # odd and even counts: lone components
    xs = [wl.random_vectors([61, n], (m, n))[0] for n, m in zip(EDGES, nx)]
    refs = [bk.apply_Ba_extended(n - 1, x, transpose=bool(transpose)) for n, x in zip(EDGES, xs)]
    mixed = _run(B, EDGES, nx, prec, np.concatenate([x.ravel() for x in xs]), transpose)
    o = 0
    for n, m, x, ref in zip(EDGES, nx, xs, refs):
        part = mixed[o:o + m * n]
        o += m * n
        assert rel_err(part.reshape(m, n), ref) <= TOL[prec], n
        # a plan of its own has other workgroups but the same arithmetic
        assert np.array_equal(_run(B, [n], [m], prec, x.ravel(), transpose), part), n
