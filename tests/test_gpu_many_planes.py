"""More (b, c, x) planes than one launch of the fused inverses takes (2^22
workgroups of 1024 threads would be 2^32 threads): both of them, t first and z
first, and the forwards of the same plans.  Every batch entry holds the same
values, so one is checked against the oracle and the others against it."""

import pytest

import oracle as O
from gpu_common import check, desc_of, dev, geometry, np_of, rand_cplx, rand_real, say, torch_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz,kz,inverse", [(2, 1, "ROWS_T_FIRST_Y"), (4, 2, "ROWS_Z_FIRST_Y")])
def test_planes_beyond_one_launch(nz, kz, inverse):
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    n, B, C = (4096, 2, nz, 5), 16, 64
    g, g1 = (geometry(n, n, (0, 0, 0, 0), (1, 1, kz), 2, b, C, C) for b in (B, 1))
    s = D.dtst_desc_schedule(desc_of(g))
    assert s.inverse == getattr(D, inverse)
    say(f"[many planes] n={n} planes={B * C * n[0]} forward={s.forward} inverse={s.inverse}")
    plan = D.Plan(desc_of(g))
    yh, x = rand_cplx((1, C) + g.K, 91), rand_real((1, C) + n, 92)
    y = torch.full((B, C) + n, float("nan"), device="cuda")
    xhat = torch.empty((B, C) + g.K, dtype=torch.complex64, device="cuda")
    plan.inverse(dev(torch, yh).expand((B, C) + g.K).contiguous(), y)
    torch.cuda.synchronize()
    check(np_of(y[:1]), O.inverse(yh, g1), "inverse, first entry")
    assert all(torch.equal(y[0], y[b]) for b in range(1, B))
    y.copy_(dev(torch, x).expand_as(y))
    plan.forward(y, xhat)
    torch.cuda.synchronize()
    check(np_of(xhat[-1:]), O.forward(x, g1), "forward, last entry")
    assert all(torch.equal(xhat[0], xhat[b]) for b in range(1, B))
    plan.close()
