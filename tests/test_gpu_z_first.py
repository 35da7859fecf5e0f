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
    "zy_shard_two_groups": ((16, 28, 87, 17), (5, 13, 3, 17), (3, 7, 70, 0), (2, 14, 10), 4, 1, 2, 1),
    "zy_shard_parts": ((2, 37, 83, 23), (2, 24, 3, 17), (0, 6, 77, 6), (1, 12, 12), 7, 1, 1, 1),
    "zy_shard_y_folded_kt7": ((2, 24, 74, 17), (2, 24, 3, 17), (0, 0, 15, 0), (1, 6, 15), 7, 1, 2, 1),
    "zy_shard_kt": ((2, 28, 62, 22), (2, 13, 3, 17), (0, 7, 43, 5), (1, 10, 11), 10, 1, 2, 1),
    "zy_shard_y_tiles_parts_kt": ((2, 25, 85, 17), (2, 24, 3, 17), (0, 0, 81, 0), (1, 12, 10), 9, 1, 2, 2),
    "zy_shard_y_folded_parts_kt": ((2, 60, 36, 17), (2, 60, 3, 17), (0, 0, 29, 0), (1, 1, 14), 9, 1, 1, 2),
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


# Whole z with y in the forward launch: (n, N_y of the shard, k_max y and z, k_t) for each of one and two t groups,
# K_t <= 8 and > 8, y unfolded and folded, ragged and whole units, and t-first rows of one and several z classes
# (whose counterparts here form shorter chains); with several units, and two tiles of modes
FUSED = [((2, 13, 8, 4), 13, 2, 3, 2), ((2, 13, 8, 4), 13, 1, 2, 3), ((2, 13, 32, 4), 13, 1, 5, 2),
         ((2, 13, 32, 4), 13, 6, 2, 3), ((2, 14, 8, 4), 14, 6, 3, 2), ((2, 16, 8, 4), 16, 1, 2, 2),
         ((2, 14, 32, 4), 14, 7, 7, 2), ((2, 14, 32, 4), 14, 5, 9, 3), ((2, 14, 17, 17), 13, 7, 5, 3),
         ((2, 15, 8, 17), 13, 6, 2, 6), ((2, 20, 64, 17), 13, 9, 7, 5), ((2, 17, 32, 17), 13, 1, 10, 8),
         ((2, 14, 17, 20), 14, 5, 3, 4), ((2, 16, 8, 20), 16, 7, 2, 7), ((2, 14, 64, 20), 14, 3, 7, 5),
         ((2, 14, 32, 20), 14, 2, 12, 3), ((2, 13, 19, 17), 13, 1, 5, 9), ((2, 13, 20, 17), 13, 5, 10, 9),
         ((2, 22, 32, 17), 13, 2, 8, 9), ((2, 13, 32, 17), 13, 1, 9, 9), ((2, 24, 18, 17), 24, 6, 2, 9),
         ((2, 26, 20, 17), 26, 13, 10, 9), ((2, 24, 32, 17), 24, 8, 8, 9), ((2, 24, 32, 17), 24, 12, 10, 9),
         ((3, 14, 64, 16), 14, 5, 8, 8), ((3, 13, 52, 16), 13, 2, 6, 5), ((2, 13, 70, 16), 13, 2, 16, 8),
         ((2, 26, 96, 12), 26, 12, 4, 5), ((2, 13, 64, 12), 13, 4, 6, 5), ((2, 14, 44, 12), 14, 4, 4, 5),
         ((2, 14, 128, 16), 14, 3, 8, 8), ((2, 40, 124, 32), 29, 14, 12, 6)]


@pytest.mark.parametrize("case", FUSED, ids=str)
def test_whole_z_fused(case):
    parity("whole z", fused_case(case), False, z_first=None)


def fused_case(case):
    n, ly, ky, kz, kt = case
    return n, (n[0], ly) + n[2:], (0, n[1] - ly, 0, 0), (1, ky, kz), kt, 1, 2, 1


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
    if z_first is None:
        assert s.forward == D.ROWS_Z_FIRST_Y and s.z_mirrored
    else:
        for way in (s.forward,) if name.startswith("zy_") or not z_first else (s.forward, s.inverse):
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
# 1.55e-7, 2.25e-7 / 1.39e-7 and 2.38e-7 / 1.50e-7.
FOUR_CLASS_ERRORS = [((32, 32, 32, 8), (8, 8, 8), 4, 1.83e-7, 1.51e-7),
                     ((16, 24, 144, 12), (8, 9, 12), 5, 1.86e-7, 1.49e-7),
                     ((16, 16, 148, 26), (6, 7, 4), 3, 2.02e-7, 1.40e-7),
                     ((24, 24, 152, 32), (5, 9, 10), 5, 2.10e-7, 1.46e-7)]


# Rows t first with even N_t below 32 and K_t > 8, unfolded, of one, two and four z classes: the same errors.  With t
# folded the forward's were 2.89e-7, 2.36e-7 and 2.52e-7; z first, at four classes, 2.35e-7 and 1.82e-7 (24 x 24 x 156).
LONG_T_ERRORS = [((32, 16, 154, 28), (6, 5, 16), 13, 2.43e-7, 1.80e-7), ((24, 24, 39, 20), (4, 10, 16), 9, 2.06e-7, 2.03e-7),
                 ((24, 64, 112, 18), (4, 6, 22), 10, 2.34e-7, 1.71e-7), ((24, 24, 156, 30), (5, 10, 28), 9, 2.18e-7, 1.81e-7)]


@pytest.mark.parametrize("n,k,kt,fwd,inv", LONG_T_ERRORS, ids=lambda v: str(v))
def test_error_with_more_than_eight_kt(n, k, kt, fwd, inv):
    import paper_2607_14394_amd as D
    assert D.dtst_desc_schedule(desc_of(geometry(n, n, (0, 0, 0, 0), k, kt, 1, 4, 4))).forward == D.ROWS_T_FIRST
    error(n, k, kt, fwd, inv)


@pytest.mark.parametrize("n,k,kt,fwd,inv", FOUR_CLASS_ERRORS, ids=lambda v: str(v))
def test_error_no_larger_than_t_first(n, k, kt, fwd, inv):
    import paper_2607_14394_amd as D
    s = D.dtst_desc_schedule(desc_of(geometry(n, n, (0, 0, 0, 0), k, kt, 1, 4, 4)))
    assert s.forward == s.inverse == D.ROWS_Z_FIRST_Y and s.z_classes == 4
    error(n, k, kt, fwd, inv)


def error(n, k, kt, fwd, inv):
    """Within 2% (the spread over inputs) of what the t-first rows are off by."""
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    g = geometry(n, n, (0, 0, 0, 0), k, kt, 1, 4, 4)
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
