"""Parity of the kernels that contract z before t (and expand t before z), on
both schedules: whole and ragged units and tiles, even and odd whole z and z
shards, one and two tiles of modes, both k_t tile counts, folded and unfolded
y with ragged slot groups, planes in parts, t shards, and more rows than a
launch keeps resident.  Every geometry needs fewer matrix instructions z first."""

import pytest

import oracle as O
from gpu_common import Guarded, check, desc_of, dev, geometry, np_of, rand_cplx, rand_real, say, torch_gpu

pytestmark = pytest.mark.gpu

# name: (n_global, n_local, offset, kmax, kt, B, C_in, C_out)
CASES = {
    "model_rows": ((2, 4, 128, 32), (2, 4, 128, 32), (0, 0, 0, 0), (1, 2, 8), 16, 1, 2, 1),
    "whole_units_nt16": ((2, 4, 64, 16), (2, 4, 64, 16), (0, 0, 0, 0), (1, 2, 8), 9, 1, 1, 2),
    "whole_units": ((2, 3, 96, 30), (2, 3, 96, 30), (0, 0, 0, 0), (1, 1, 13), 11, 1, 2, 2),
    "two_mode_tiles_kt8": ((2, 3, 101, 32), (2, 3, 101, 32), (0, 0, 0, 0), (1, 1, 16), 8, 1, 1, 1),
    "two_mode_tiles": ((2, 3, 99, 9), (2, 3, 99, 9), (0, 0, 0, 0), (1, 1, 23), 5, 1, 2, 1),
    "full_spectrum": ((2, 2, 30, 30), (2, 2, 30, 30), (0, 0, 0, 0), (1, 1, 15), 16, 1, 1, 1),
    "one_t_group": ((2, 3, 75, 10), (2, 3, 75, 10), (0, 0, 0, 0), (1, 1, 11), 6, 1, 2, 1),
    "odd_z": ((2, 2, 33, 21), (2, 2, 33, 21), (0, 0, 0, 0), (1, 1, 7), 11, 1, 1, 1),
    "z_shard": ((2, 2, 64, 32), (2, 2, 23, 32), (0, 0, 17, 0), (1, 1, 8), 16, 1, 1, 2),
    "t_shard": ((2, 2, 32, 40), (2, 2, 32, 13), (0, 0, 0, 9), (1, 1, 6), 12, 2, 1, 1),
    "few_z": ((2, 2, 5, 32), (2, 2, 3, 32), (0, 0, 1, 0), (1, 1, 2), 10, 1, 1, 1),
    "y_unfolded_groups": ((3, 37, 40, 32), (3, 37, 40, 32), (0, 0, 0, 0), (1, 9, 5), 9, 1, 2, 1),
    "y_shard": ((3, 80, 40, 30), (3, 40, 40, 30), (0, 11, 0, 0), (1, 16, 4), 16, 1, 1, 2),
    "y_folded_parts": ((4, 112, 48, 32), (2, 112, 48, 32), (1, 0, 0, 0), (2, 8, 6), 16, 1, 2, 3),
    "x_folded_parts": ((8, 96, 64, 30), (8, 96, 64, 30), (0, 0, 0, 0), (3, 4, 7), 10, 1, 1, 1),
    "many_rows": ((33, 80, 20, 20), (33, 80, 20, 20), (0, 0, 0, 0), (3, 9, 4), 10, 1, 2, 2),
}


@pytest.mark.parametrize("split", [False, True], ids=["default", "split"])
@pytest.mark.parametrize("name", list(CASES))
def test_z_first(name, split):
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    g = geometry(*CASES[name])
    say(f"[z first {name}] n_local={g.n_local} kmax={g.kmax} kt={g.kt} split={split}")
    plan = D.Plan(desc_of(g), flags=D.PLAN_SPLIT_SCHEDULE if split else 0)
    x, gy = rand_real((g.batch, g.c_in) + g.n_local, 71), rand_real((g.batch, g.c_out) + g.n_local, 72)
    yh, gxh = rand_cplx((g.batch, g.c_out) + g.K, 73), rand_cplx((g.batch, g.c_in) + g.K, 74)
    xhat = Guarded(torch, plan.spectral_shape(g.c_in), torch.complex64)
    gyh = Guarded(torch, plan.spectral_shape(g.c_out), torch.complex64)
    y = Guarded(torch, plan.spatial_shape(g.c_out), torch.float32)
    gx = Guarded(torch, plan.spatial_shape(g.c_in), torch.float32)
    plan.forward(dev(torch, x), xhat.t)
    plan.forward(dev(torch, x), xhat.t, accumulate=True)
    plan.inverse_adj(dev(torch, gy), gyh.t)
    plan.inverse(dev(torch, yh), y.t)
    plan.forward_adj(dev(torch, gxh), gx.t)
    torch.cuda.synchronize()
    check(np_of(xhat.t), 2 * O.forward(x, g), "forward + accumulate")
    check(np_of(gyh.t), O.inverse_adj(gy, g), "inverse_adj")
    check(np_of(y.t), O.inverse(yh, g), "inverse")
    check(np_of(gx.t), O.forward_adj(gxh, g), "forward_adj")
    for b in (xhat, gyh, y, gx):
        assert b.guards_intact()
    plan.close()
