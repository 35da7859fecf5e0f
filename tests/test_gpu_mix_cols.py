"""Parity of the mix, its data gradient and the weight gradient (overwriting
and accumulating) at channel counts around the column forms: odd and even
C_out, wave-filling and ragged lane counts, one to several chunks of rows, the
widest column form and the row-group form behind it, mode ranges that do not
fill a block, and guard bands."""

import numpy as np
import pytest

from gpu_common import Guarded, check, desc_of, dev, geometry, np_of, rand_cplx, say, torch_gpu

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 1), (2, 3, 2), (1, 5, 5), (1, 20, 20), (3, 4, 6), (2, 21, 9), (1, 33, 17), (1, 32, 32), (2, 7, 48),
         (1, 13, 63), (2, 3, 64), (1, 2, 66), (1, 13, 14), (2, 20, 12), (3, 17, 18), (3, 20, 3), (3, 13, 13),
         (2, 17, 31), (3, 5, 7), (2, 4, 63)]


@pytest.mark.parametrize("b,ci,co", CASES)
def test_mix_and_gradients(b, ci, co):
    parity((6, 8, 8, 8), (2, 3, 3), 3, b, ci, co, lambda M: ((0, M), (5, 5 + 137), (M - 1, M)))


@pytest.mark.parametrize("b,ci,co", [c for c in CASES if c[0] > 1 and c[2] <= 64] + [(2, 10, 29), (3, 28, 28), (2, 6, 26)])
def test_columns_of_several_batch_entries(b, ci, co):
    """Column forms with B > 1, which take over from the row groups at 256 blocks of 4 x 64 / (C_out / W) modes: one
    block fewer, and that many with a ragged last one."""
    modes = 4 * (64 // (co // (2 if co % 2 == 0 else 1)))
    parity((32, 32, 16, 8), (16, 16, 8), 5, b, ci, co,
           lambda M: ((6, 6 + 255 * modes), (6, 6 + 255 * modes + 1), (7, 7 + 128 * modes + 1)))


def parity(n, k, kt, b, ci, co, ranges):
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    g = geometry(n, n, (0, 0, 0, 0), k, kt, b, ci, co)
    plan = D.Plan(desc_of(g))
    M = plan.n_modes
    for m0, m1 in ranges(M):
        say(f"[mix columns] B={b} {ci}->{co} modes [{m0}, {m1})")
        x, gy = rand_cplx((b, ci) + g.K, 81), rand_cplx((b, co) + g.K, 82)
        w, g0 = rand_cplx((m1 - m0, ci, co), 83), rand_cplx((m1 - m0, ci, co), 84)
        y = Guarded(torch, plan.spectral_shape(co), torch.complex64, fill=torch.zeros(()).cuda())
        gx = Guarded(torch, plan.spectral_shape(ci), torch.complex64, fill=torch.zeros(()).cuda())
        gw = Guarded(torch, w.shape, torch.complex64)
        ga = Guarded(torch, w.shape, torch.complex64, fill=dev(torch, g0))
        plan.mix(dev(torch, x), dev(torch, w), y.t, m0, m1)
        plan.mix(dev(torch, gy), dev(torch, w), gx.t, m0, m1, op=1)
        plan.wgrad(dev(torch, x), dev(torch, gy), gw.t, m0, m1)
        plan.wgrad(dev(torch, x), dev(torch, gy), ga.t, m0, m1, accumulate=True)
        torch.cuda.synchronize()
        xs = x.reshape(b, ci, M)[:, :, m0:m1].astype(np.complex128)
        gs = gy.reshape(b, co, M)[:, :, m0:m1].astype(np.complex128)
        wd = w.astype(np.complex128)
        ref_y, ref_gx = np.zeros((b, co, M), np.complex128), np.zeros((b, ci, M), np.complex128)
        ref_y[:, :, m0:m1] = np.einsum("bim,mio->bom", xs, wd)
        ref_gx[:, :, m0:m1] = np.einsum("bom,mio->bim", gs, wd.conj())
        ref_gw = np.einsum("bim,bom->mio", xs.conj(), gs)
        check(np_of(y.t).reshape(b, co, M), ref_y, "mix")
        check(np_of(gx.t).reshape(b, ci, M), ref_gx, "data gradient")
        check(np_of(gw.t), ref_gw, "weight gradient")
        check(np_of(ga.t), ref_gw + g0, "weight gradient, accumulated")
        for t in (y, gx, gw, ga):
            assert t.guards_intact()
    plan.close()
