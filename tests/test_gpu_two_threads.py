"""Two plans on two host threads and streams, one of the longest and one of the shortest lengths
of each kernel with a run-time LDS size (whole products in LDS, chirp convolutions, the
one-launch P^{-1} scan): every call succeeds and every result has the bits of a run alone."""

import threading

import numpy as np
import pytest

from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dev

pytestmark = pytest.mark.gpu

CALLS = 400


def _worker(B, plan, stream, what, v, J, calls, outs, errs):
    import torch
    try:
        with torch.cuda.stream(stream):
            for k in range(calls):
                o = outs[k % len(outs)]
                if what == "pinv":
                    B.birk_precond(plan, J, v, o, 1, B.BIRK_J_CONSTANT)
                else:
                    B.birk_apply(plan, v, o)
        stream.synchronize()
    except Exception as e:   # noqa: BLE001 -- handed to the main thread
        errs.append(e)


#         LDS products: M = 4096 against 16 | chirp: longest rows and columns against the shortest | scans of 4 waves against 1
@pytest.mark.parametrize("what,long,short", [("lds", (1366, 6), (6, 6)), ("lds", (2049, 6), (9, 6)),
                                             ("chirp", (1000000, 2), (1367, 6)), ("pinv", (256, 8), (17, 8))])
def test_long_and_short_side_by_side(what, long, short):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    announce(f"two threads {what} {long} {short}")
    jobs = []
    for k, (Nn, nx) in enumerate((long, short)):
        st = torch.cuda.Stream()
        v = dev(wl.random_vectors([94, k], (Nn * nx,))[0], torch.float64)
        J = dev(wl.lti_matrix(np.random.default_rng([95, k]), nx).ravel(), torch.float64)
        torch.cuda.synchronize()
        plan = B.birk_plan_create([Nn], [nx], B.BIRK_F64, stream=st)
        alone = torch.empty_like(v)
        outs = [torch.empty_like(v) for _ in range(4)]
        errs = []
        _worker(B, plan, st, what, v, J, 1, [alone], errs)
        assert not errs
        jobs.append((plan, st, v, J, alone, outs, errs))
    torch.cuda.synchronize()
    ths = [threading.Thread(target=_worker, args=(B, p, st, what, v, J, CALLS, outs, errs))
           for p, st, v, J, _, outs, errs in jobs]
    for t in ths:
        t.start()
    for t in ths:
        t.join()
    torch.cuda.synchronize()
    for plan, _, _, _, alone, outs, errs in jobs:
        assert not errs, errs
        for o in outs:
            assert torch.equal(o, alone)
        plan.destroy()
