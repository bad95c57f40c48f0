"""GPU parity of the even chirp convolutions (any N whose transforms do not fit one workgroup)
where their length changes: M = 4N exactly for M = 3, 4, 5 times a power of two, one node
either side of it, and the first N of the path; alone and mixed in one plan, whose launches
then hold tiles of every kind.  Reference: the oracle's extended-precision product; bars as
in the product tests (1e-12, 2e-5, 1e-13 relative to the largest value).  Then each two-step
split the tuner may choose, through a tuned plan of every length class, against the untuned
one (1e-13: the bar of the other tuner tests)."""

import numpy as np
import pytest

from oracle import birkhoff as bk
from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dev, from_df32, host, rel_err, to_df32

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 2e-5, "df32": 1e-13}
#   first N | 4N = 3 2^11 -1, 0, +1 | = 2^13 -1, +1 | = 5 2^11 -1, 0, +1 | = 3 2^12 -1, 0, +1
NS = [1366, 1535, 1536, 1537, 2047, 2049, 2559, 2560, 2561, 3071, 3072, 3073]


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk
    return birk


def _run(B, Nn, nx, prec, x, transpose):
    import torch
    plan = B.birk_plan_create(Nn, nx, {"f64": B.BIRK_F64, "f32": B.BIRK_F32, "df32": B.BIRK_DF32}[prec])
    v = dev(to_df32(x[None, :])[0]) if prec == "df32" else dev(x, torch.float64 if prec == "f64" else torch.float32)
    out = torch.full_like(v, float("nan"))
    (B.birk_apply_T if transpose else B.birk_apply)(plan, v, out)
    torch.cuda.synchronize()
    r = host(out)
    plan.destroy()
    return from_df32(r[None, :])[0] if prec == "df32" else r.astype(np.float64)


@pytest.mark.parametrize("prec", ["f64", "f32", "df32"])
@pytest.mark.parametrize("transpose", [0, 1])
def test_length_edges_alone_and_mixed(B, prec, transpose):
    announce(f"chirp convolutions {prec} transpose={transpose}")
    Nn = [n + 1 for n in NS]
    nx = [1 + i % 3 for i in range(len(NS))]
    xs = [wl.random_vectors([71, n], (m, n))[0] for n, m in zip(Nn, nx)]
    mixed = _run(B, Nn, nx, prec, np.concatenate([x.ravel() for x in xs]), transpose)
    o = 0
    for n, m, x in zip(Nn, nx, xs):
        part = mixed[o:o + m * n]
        o += m * n
        ref = bk.apply_Ba_extended(n - 1, x, transpose=bool(transpose))
        assert rel_err(part.reshape(m, n), ref) <= TOL[prec], n
        assert np.array_equal(_run(B, [n], [m], prec, x.ravel(), transpose), part), n


@pytest.mark.parametrize("base", [3, 4, 5, 6])
def test_every_split_of_every_class(B, base):
    """N just under base 2^k / 4 for every class 2^13..2^20 of one plan: tuning runs every
    split of every class; whatever it keeps must give the untuned products."""
    import torch
    Nns = [(base << k) // 4 for k in range(11, 18)]     # N = Nn - 1: 4N just under base 2^k
    Nns = [n for n in Nns if n > 1400]
    announce(f"chirp splits N_n {Nns}")
    x = wl.random_vectors([72, base], (sum(Nns),))[0]
    plan = B.birk_plan_create(Nns, [1] * len(Nns), B.BIRK_F64)
    v = dev(x, torch.float64)

    def both():
        outs = []
        for f in (B.birk_apply, B.birk_apply_T):
            out = torch.full_like(v, float("nan"))
            f(plan, v, out)
            torch.cuda.synchronize()
            outs.append(host(out))
        return outs

    before = both()
    rep = B.birk_plan_tune(plan)
    after = both()
    plan.destroy()
    assert rep.count(" chosen [M1 2^") == len(Nns)
    for a, b in zip(after, before):
        assert rel_err(a, b) <= 1e-13
