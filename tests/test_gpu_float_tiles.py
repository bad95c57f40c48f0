"""Float products of N a power of two in tiles of sixteen columns, which batches of components
take from four workgroups a CU: at each length of the path, at that batch size and one
component below it.  A few components against the oracle's extended-precision product (2e-5 of
the largest value, the bar of the float products); all of them bit for bit against the same
components in plans of six, whose tiles hold eight columns."""

import numpy as np
import pytest

from oracle import birkhoff as bk
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("transpose", [0, 1])
@pytest.mark.parametrize("logN,nc", [(15, 114), (16, 61), (17, 61), (18, 32)])
def test_sixteen_columns(logN, nc, transpose):
    import torch
    assert torch.cuda.is_available()
    from paper_2509_01855_amd import birk as B
    N = 1 << logN
    announce(f"float tiles N=2^{logN} nc={nc} transpose={transpose}")
    x = np.random.default_rng([logN, 7]).standard_normal((nc, N + 1)).astype(np.float32)

    def run(rows):
        plan = B.birk_plan_create([N + 1], [len(rows)], B.BIRK_F32)
        v = torch.from_numpy(np.ascontiguousarray(rows).ravel()).cuda()
        out = torch.full_like(v, float("nan"))
        (B.birk_apply_T if transpose else B.birk_apply)(plan, v, out)
        torch.cuda.synchronize()
        plan.destroy()
        return out.cpu().numpy().reshape(rows.shape)

    full, below = run(x), run(x[:nc - 1])
    assert np.array_equal(full[:nc - 1], below)
    for c in range(0, nc, 6):
        assert np.array_equal(run(x[c:c + 6]), full[c:c + 6]), c
    for k in (0, 1, N // 3, N // 2, N - 1, N):
        w = bk.ba_col(N, k) if transpose else bk.ba_row(N, k)
        ref = x.astype(np.float64) @ w
        assert np.max(np.abs(full[:, k] - ref)) <= 2e-5 * np.max(np.abs(full)), k
