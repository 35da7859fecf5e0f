"""Parity at t extents that are not whole 16-byte chunks: a row's last t chunk
then starts early (its values overlap the previous chunk's), rows lie at any
4-byte alignment, and the t fold of k_t > 8 splits an even extent at any
position.  Extents at the edges of the t groups (16, 32), every remainder mod
4, folded and unfolded z, ragged z tiles, both schedules; the fused inverse +
block epilogue at even extents; the point-wise layer at point counts that are
not multiples of 4."""

import numpy as np
import pytest

import oracle as O
from gpu_common import Guarded, check, desc_of, dev, geometry, np_of, rand_cplx, rand_real, say, torch_gpu

pytestmark = pytest.mark.gpu

# (N_t, k_t): below one chunk, one chunk, each remainder, around the 16- and 32-wide groups
EXTENTS = [(3, 2), (4, 3), (5, 3), (6, 2), (7, 4), (13, 7), (15, 8), (17, 5), (17, 9), (18, 10), (19, 10), (21, 11),
           (22, 12), (26, 9), (30, 16), (31, 8), (31, 16), (33, 6), (34, 16), (47, 3), (63, 13)]
# (N_x, N_y, N_z), k_max of z: folded whole tiles, folded ragged tile, odd N_z
GRIDS = [((3, 4, 32), 5), ((2, 6, 26), 3), ((3, 5, 19), 7)]


# Long z whose folded t image would not fit the LDS: t stays unfolded
LONG_Z = [((2, 3, 976, 26), 7, 12), ((3, 2, 303, 20), 22, 10), ((2, 2, 232, 18), 52, 10), ((2, 2, 314, 24), 62, 11)]


@pytest.mark.parametrize("split", [False, True], ids=["default", "split"])
@pytest.mark.parametrize("n,kz,kt", LONG_Z, ids=lambda v: str(v[2:]) if isinstance(v, tuple) else str(v))
def test_long_z(n, kz, kt, split):
    transforms([(n[:3], kz)], n[3], kt, split)


@pytest.mark.parametrize("split", [False, True], ids=["default", "split"])
@pytest.mark.parametrize("nt,kt", EXTENTS)
def test_transforms(nt, kt, split):
    transforms(GRIDS, nt, kt, split)


def transforms(grids, nt, kt, split):
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    for (nx, ny, nz), kz in grids:
        n = (nx, ny, nz, nt)
        g = geometry(n, n, (0, 0, 0, 0), (1, min(2, ny // 2), kz), kt, 2, 3, 2)
        say(f"[t chunks] n={n} kt={kt} kz={kz} split={split}")
        plan = D.Plan(desc_of(g), flags=D.PLAN_SPLIT_SCHEDULE if split else 0)
        x, gy = rand_real((2, 3) + n, 41), rand_real((2, 2) + n, 42)
        yh, gxh = rand_cplx((2, 2) + g.K, 43), rand_cplx((2, 3) + g.K, 44)
        xhat = Guarded(torch, plan.spectral_shape(3), torch.complex64)
        gyh = Guarded(torch, plan.spectral_shape(2), torch.complex64)
        y = Guarded(torch, plan.spatial_shape(2), torch.float32)
        gx = Guarded(torch, plan.spatial_shape(3), torch.float32)
        plan.forward(dev(torch, x), xhat.t)
        plan.inverse_adj(dev(torch, gy), gyh.t)
        plan.inverse(dev(torch, yh), y.t)
        plan.forward_adj(dev(torch, gxh), gx.t)
        torch.cuda.synchronize()
        check(np_of(xhat.t), O.forward(x, g), "forward")
        check(np_of(gyh.t), O.inverse_adj(gy, g), "inverse_adj")
        check(np_of(y.t), O.inverse(yh, g), "inverse")
        check(np_of(gx.t), O.forward_adj(gxh, g), "forward_adj")
        for b in (xhat, gyh, y, gx):
            assert b.guards_intact()
        plan.close()


@pytest.mark.parametrize("c", [3, 16, 20, 32])
@pytest.mark.parametrize("nt,kt", [(6, 3), (18, 10), (20, 9), (20, 6), (22, 5), (24, 11), (26, 12), (28, 9), (30, 7),
                                   (30, 16)])
def test_inverse_block(nt, kt, c):
    """Even extents: the fused kernel (whole and ragged last z tiles) with each channel class; t folded (K_t > 8) with
    halves that are whole 16-byte chunks (24) and that are not (18, 20, 22, 26, 28, 30)."""
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    for nz, kz in ((32, 5), (26, 3) if nt % 4 == 0 else (20, 3)):
        n = (2, 3, nz, nt)
        g = geometry(n, n, (0, 0, 0, 0), (1, 1, kz), kt, 2, c, c)
        say(f"[t chunks, block] n={n} kt={kt} c={c}")
        plan = D.Plan(desc_of(g))
        assert plan.block_fused == 1
        yh, x = rand_cplx((2, c) + g.K, 51), rand_real((2, c) + n, 52)
        wb = (rand_real((c, c), 53) / np.sqrt(c)).astype(np.float32)
        y = Guarded(torch, plan.spatial_shape(c), torch.float32)
        plan.inverse_block(dev(torch, yh), dev(torch, x), dev(torch, wb), y.t)
        torch.cuda.synchronize()
        check(np_of(y.t), O.block_epilogue(x, wb, O.inverse(yh, g)), "inverse + block epilogue")
        assert y.guards_intact()
        plan.close()


@pytest.mark.parametrize("n,kz,kt,c", [((2, 3, 288, 28), 8, 15, 20), ((2, 2, 388, 28), 5, 13, 20),
                                       ((2, 2, 386, 28), 10, 11, 16), ((2, 2, 480, 28), 8, 9, 32)])
def test_inverse_block_long_z(n, kz, kt, c):
    """t does not fold in the fused block kernel where its LDS does not hold the folded z image."""
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    g = geometry(n, n, (0, 0, 0, 0), (1, 1, kz), kt, 2, c, c)
    s = D.dtst_desc_schedule(desc_of(g))
    assert s.block == D.BLOCK_CHUNKS and not s.block_t_folded
    say(f"[t chunks, long block] n={n} kt={kt} c={c}")
    plan = D.Plan(desc_of(g))
    yh, x = rand_cplx((2, c) + g.K, 51), rand_real((2, c) + n, 52)
    wb = (rand_real((c, c), 53) / np.sqrt(c)).astype(np.float32)
    y = Guarded(torch, plan.spatial_shape(c), torch.float32)
    plan.inverse_block(dev(torch, yh), dev(torch, x), dev(torch, wb), y.t)
    torch.cuda.synchronize()
    check(np_of(y.t), O.block_epilogue(x, wb, O.inverse(yh, g)), "inverse + block epilogue")
    assert y.guards_intact()
    plan.close()


@pytest.mark.parametrize("points", [1, 3, 4, 5, 6, 7, 1022])
def test_pointwise_and_epilogue(points):
    """Point counts around the 4-point accesses; in place (epilogue) and out of place (point-wise layer)."""
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    ci, co, batch = 5, 18, 3
    x, w, b = rand_real((batch, ci, points), 61), rand_real((co, ci), 62), rand_real((co,), 63)
    y = Guarded(torch, (batch, co, points), torch.float32)
    D.dtst_pointwise(dev(torch, x), dev(torch, w), dev(torch, b), y.t, act=1)
    torch.cuda.synchronize()
    check(np_of(y.t), O.pointwise(x, w, b, act=True), "pointwise")
    assert y.guards_intact()
    n = (1, 1, 1, points) if points < 64 else (1, 1, 73, 14)
    g = geometry((2, 2, max(n[2], 2), n[3]), n, (0, 0, 0, 0), (1, 1, 1), 1, batch, ci, co)
    plan = D.Plan(desc_of(g))
    x, y0 = rand_real((batch, ci) + n, 64), rand_real((batch, co) + n, 65)
    y = Guarded(torch, (batch, co) + n, torch.float32)
    y.t.copy_(dev(torch, y0))
    plan.block_epilogue(dev(torch, x), dev(torch, w), y.t)
    torch.cuda.synchronize()
    check(np_of(y.t), O.block_epilogue(x, w, y0), "block epilogue")
    assert y.guards_intact()
    plan.close()


@pytest.mark.parametrize("c", [14, 24])
@pytest.mark.parametrize("nt,nz", [(4, 17), (4, 111), (6, 24), (6, 50), (6, 64), (8, 40), (8, 75), (8, 137), (12, 35),
                                   (12, 60), (16, 90), (16, 112)])
def test_inverse_block_z_runs(nt, nz, c):
    """One t group, one z class: chunks of one, two and four z tiles, whole and ragged last ones and rows of fewer."""
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    n = (2, 3, nz, nt)
    g = geometry(n, n, (0, 0, 0, 0), (1, 1, 5), 3, 2, c, c)
    assert D.dtst_desc_schedule(desc_of(g)).block == D.BLOCK_CHUNKS
    say(f"[t chunks, z runs] n={n} c={c}")
    plan = D.Plan(desc_of(g))
    yh, x = rand_cplx((2, c) + g.K, 51), rand_real((2, c) + n, 52)
    wb = (rand_real((c, c), 53) / np.sqrt(c)).astype(np.float32)
    y = Guarded(torch, plan.spatial_shape(c), torch.float32)
    plan.inverse_block(dev(torch, yh), dev(torch, x), dev(torch, wb), y.t)
    torch.cuda.synchronize()
    check(np_of(y.t), O.block_epilogue(x, wb, O.inverse(yh, g)), "inverse + block epilogue")
    assert y.guards_intact()
    plan.close()


# (n, k_max z, k_t, C_in, C_out, shard): row tasks of few input channels
ROW_BLOCKS = [((2, 3, 204, 16), 19, 4, 5, 5, None), ((3, 7, 27, 8), 13, 3, 4, 4, None),
              ((2, 5, 36, 32), 13, 5, 7, 7, None), ((2, 3, 50, 30), 8, 16, 8, 32, None),
              ((2, 3, 31, 8), 9, 3, 12, 3, None), ((2, 2, 40, 12), 16, 7, 1, 2, (9, 17)), ((5, 61, 2, 6), 1, 2, 3, 1, None),
              ((9, 40, 50, 32), 6, 9, 2, 5, None)]


# few input channels, and rows too short for their output channels to be row tasks: chunks
SHORT_ROWS = [((4, 13, 16, 32), 7, 7, 8, 30, None), ((3, 11, 20, 10), 8, 4, 9, 32, None),
              ((4, 7, 14, 20), 5, 7, 4, 20, None), ((2, 9, 16, 8), 5, 3, 1, 32, None),
              ((2, 9, 25, 12), 4, 3, 6, 17, (11, 9)), ((2, 3, 30, 30), 8, 16, 8, 32, None),
              ((3, 5, 38, 32), 10, 10, 5, 16, None), ((3, 5, 38, 32), 10, 5, 5, 16, None)]


@pytest.mark.parametrize("case", ROW_BLOCKS + SHORT_ROWS, ids=lambda c: "x".join(map(str, c[0])) + f"_c{c[3]}_{c[4]}")
def test_inverse_block_few_channels(case):
    """One to three tiles of input channels, one and two mode tiles, ragged and few z positions, a z shard, fewer
    and more rows than a launch keeps resident."""
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    ng, kz, kt, ci, co, shard = case
    off, nz = shard if shard else (0, ng[2])
    n = (ng[0], ng[1], nz, ng[3])
    g = geometry(ng, n, (0, 0, off, 0), (1, 1, kz), kt, 2, ci, co)
    say(f"[row block] n={n} kz={kz} kt={kt} c={ci}->{co}")
    plan = D.Plan(desc_of(g))
    yh, x = rand_cplx((2, co) + g.K, 55), rand_real((2, ci) + n, 56)
    wb = (rand_real((co, ci), 57) / np.sqrt(ci)).astype(np.float32)
    y = Guarded(torch, plan.spatial_shape(co), torch.float32)
    plan.inverse_block(dev(torch, yh), dev(torch, x), dev(torch, wb), y.t)
    torch.cuda.synchronize()
    check(np_of(y.t), O.block_epilogue(x, wb, O.inverse(yh, g)), "inverse + block epilogue")
    assert y.guards_intact()
    plan.close()
