"""The tuner tries every pass-A/C tile width that a group's type, length and component count
distinguish: 61 float components at N = 2^16 give the sixteen-column tiles their four workgroups
a CU at L1 = 2^8, where eight columns (narrow) are another schedule, and 59 do not.  The tuned
products against the untuned ones: 2e-6 (rounding order only), as in the other tuner tests."""

import numpy as np
import pytest

from paper_2509_01855_amd import workloads as wl
from tests.gpu_util import announce, dev, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,wide", [(61, True), (59, False)])
def test_narrow_candidates_of_float_groups(nx, wide):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    Nn = (1 << 16) + 1
    announce(f"tuner widths, {nx} float components of 2^16 + 1 nodes")
    plan = B.birk_plan_create([Nn], [nx], B.BIRK_F32)
    v = dev(wl.random_vectors([96, nx], (nx * Nn,))[0], torch.float32)
    outs = []
    for tuned in (0, 1):
        if tuned:
            rep = B.birk_plan_tune(plan)
        out = torch.full_like(v, float("nan"))
        B.birk_apply(plan, v, out)
        torch.cuda.synchronize()
        outs.append(host(out).astype(np.float64))
    plan.destroy()
    cand = rep[:rep.index("chosen")]
    assert ("[split 0, tb 2, xcd 1, streams 1, narrow 1]" in cand) == wide
    assert "[split 1, tb 2, xcd 1, streams 1, narrow 1]" in cand   # L1 = 2^9: eight or four columns
    assert rel_err(outs[1], outs[0]) <= 2e-6
