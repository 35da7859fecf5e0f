"""Parity of the kernels that contract z before t (and expand t before z), on
both schedules: whole and ragged units and tiles, even and odd whole z and z
shards, one and two tiles of modes, both k_t tile counts, folded and unfolded
y with ragged slot groups, planes in parts, t shards, and more rows than a
launch keeps resident.  Every geometry of CASES goes z first (asserted from the
library's schedule); those of T_FIRST are their neighbours that fold t and stay
t first."""

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
    "full_spectrum": ((2, 2, 30, 29), (2, 2, 30, 29), (0, 0, 0, 0), (1, 1, 15), 15, 1, 1, 1),
    "one_t_group": ((2, 3, 75, 10), (2, 3, 75, 10), (0, 0, 0, 0), (1, 1, 11), 6, 1, 2, 1),
    "odd_z": ((2, 2, 33, 21), (2, 2, 33, 21), (0, 0, 0, 0), (1, 1, 7), 11, 1, 1, 1),
    "z_shard": ((2, 2, 64, 31), (2, 2, 23, 31), (0, 0, 17, 0), (1, 1, 8), 16, 1, 1, 2),
    "t_shard": ((2, 2, 32, 40), (2, 2, 32, 13), (0, 0, 0, 9), (1, 1, 6), 12, 2, 1, 1),
    "few_z": ((2, 2, 5, 16), (2, 2, 2, 16), (0, 0, 3, 0), (1, 1, 1), 9, 1, 1, 1),
    "y_unfolded_groups": ((3, 37, 40, 32), (3, 37, 40, 32), (0, 0, 0, 0), (1, 9, 5), 9, 1, 2, 1),
    "y_shard": ((3, 80, 40, 30), (3, 40, 40, 30), (0, 11, 0, 0), (1, 16, 4), 16, 1, 1, 2),
    "y_folded_parts": ((4, 112, 48, 32), (2, 112, 48, 32), (1, 0, 0, 0), (2, 8, 6), 16, 1, 2, 3),
    "x_folded_parts": ((8, 96, 64, 30), (8, 96, 64, 30), (0, 0, 0, 0), (3, 4, 7), 10, 1, 1, 1),
    "many_rows": ((33, 80, 20, 21), (33, 80, 20, 21), (0, 0, 0, 0), (3, 9, 4), 10, 1, 4, 4),
    # z shards with y in the forward launch: one and two t groups, K_t <= 8 and > 8, y folded, unfolded and a shard,
    # one and two y tiles, planes in parts (their inverses may stay t first)
    "zy_shard_one_group": ((16, 29, 56, 16), (16, 29, 41, 16), (0, 0, 0, 0), (2, 11, 4), 8, 1, 1, 2),
    "zy_shard_y_folded": ((2, 60, 38, 8), (2, 60, 26, 8), (0, 0, 12, 0), (1, 16, 2), 1, 2, 2, 1),
    "zy_shard_two_groups": ((16, 10, 214, 32), (5, 7, 22, 32), (3, 1, 150, 0), (2, 1, 10), 3, 1, 2, 1),
    "zy_shard_parts": ((2, 19, 79, 23), (2, 19, 2, 23), (0, 0, 31, 0), (1, 2, 10), 9, 1, 1, 1),
    "zy_shard_y_folded_parts": ((2, 34, 36, 33), (2, 34, 2, 26), (0, 0, 6, 5), (1, 12, 10), 9, 1, 1, 2),
    "zy_shard_y_tiles_parts": ((2, 32, 22, 27), (2, 18, 2, 27), (0, 7, 10, 0), (1, 9, 9), 11, 1, 2, 2),
    "zy_shard_y_folded_parts_kt2": ((2, 34, 61, 31), (2, 34, 2, 17), (0, 0, 9, 0), (1, 7, 10), 2, 1, 1, 1),
    # z shards of whole rows of 32, two mode tiles, two k_t tiles, the whole z spectrum: y in launches of its own
    "shard_t32": ((2, 19, 20, 32), (2, 2, 17, 32), (0, 16, 2, 0), (1, 5, 9), 4, 1, 2, 1),
    "rows_shard_two_tiles": ((2, 65, 38, 32), (2, 65, 36, 32), (0, 0, 2, 0), (1, 4, 19), 7, 1, 1, 2),
    "rows_shard_kt": ((2, 8, 43, 38), (2, 2, 18, 26), (0, 3, 3, 4), (1, 1, 21), 15, 1, 1, 1),
    "rows_shard_full": ((2, 2, 62, 29), (2, 2, 22, 19), (0, 0, 29, 7), (1, 1, 31), 15, 1, 1, 1),
}

T_FIRST = {
    "full_spectrum": ((2, 2, 30, 30), (2, 2, 30, 30), (0, 0, 0, 0), (1, 1, 15), 16, 1, 1, 1),
    "z_shard": ((2, 2, 64, 32), (2, 2, 23, 32), (0, 0, 17, 0), (1, 1, 8), 16, 1, 1, 2),
    "few_z": ((2, 2, 5, 32), (2, 2, 3, 32), (0, 0, 1, 0), (1, 1, 2), 10, 1, 1, 1),
    "many_rows": ((33, 80, 20, 20), (33, 80, 20, 20), (0, 0, 0, 0), (3, 9, 4), 10, 1, 2, 2),
}


@pytest.mark.parametrize("split", [False, True], ids=["default", "split"])
@pytest.mark.parametrize("name", list(CASES))
def test_z_first(name, split):
    parity(name, CASES[name], split, z_first=True)


@pytest.mark.parametrize("name", list(T_FIRST))
def test_t_first_neighbours(name):
    parity(name, T_FIRST[name], False, z_first=False)


def parity(name, case, split, z_first):
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    g = geometry(*case)
    flags = D.PLAN_SPLIT_SCHEDULE if split else 0
    s = D.dtst_desc_schedule(desc_of(g), flags)
    say(f"[z first {name}] n_local={g.n_local} kmax={g.kmax} kt={g.kt} split={split} forward={s.forward} "
        f"inverse={s.inverse}")
    for way in (s.forward,) if name.startswith("zy_") else (s.forward, s.inverse):
        assert (way >= D.ROWS_Z_FIRST) == z_first
    plan = D.Plan(desc_of(g), flags=flags)
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


# n, kmax, kt, the error of the t-first rows with z in four classes on such inputs: relative L2 of forward and inverse
# against 64 bits (N(0, 1) fields and spectra).  z first without the shorter chains: 1.94e-7 / 1.58e-7, 2.16e-7 /
# 1.55e-7 and 2.25e-7 / 1.39e-7.
FOUR_CLASS_ERRORS = [((32, 32, 32, 8), (8, 8, 8), 4, 1.83e-7, 1.51e-7),
                     ((16, 24, 144, 12), (8, 9, 12), 5, 1.86e-7, 1.49e-7),
                     ((16, 16, 148, 26), (6, 7, 4), 3, 2.02e-7, 1.40e-7)]


@pytest.mark.parametrize("n,k,kt,fwd,inv", FOUR_CLASS_ERRORS, ids=lambda v: str(v))
def test_error_no_larger_than_t_first(n, k, kt, fwd, inv):
    """Within 2% (the spread over inputs) of what the t-first rows are off by."""
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    g = geometry(n, n, (0, 0, 0, 0), k, kt, 1, 4, 4)
    s = D.dtst_desc_schedule(desc_of(g))
    assert s.forward == s.inverse == D.ROWS_Z_FIRST_Y and s.z_classes == 4
    say(f"[z first error] n={n} kmax={k} kt={kt}")
    plan = D.Plan(desc_of(g))
    x, yh = rand_real((1, 4) + n, 75), rand_cplx((1, 4) + g.K, 76)
    xhat = torch.empty(plan.spectral_shape(4), dtype=torch.complex64, device="cuda")
    y = torch.empty(plan.spatial_shape(4), device="cuda")
    plan.forward(dev(torch, x), xhat)
    plan.inverse(dev(torch, yh), y)
    torch.cuda.synchronize()
    check(np_of(xhat), O.forward(x, g), "forward", rel_l2=1.02 * fwd)
    check(np_of(y), O.inverse(yh, g), "inverse", rel_l2=1.02 * inv)
    plan.close()
