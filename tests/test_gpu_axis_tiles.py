"""Parity of the separate y contraction where its columns (K_z K_t) are not
whole work items: the waves' 16- and 32-column tiles of all (b, c, x) then run
on in one sequence, items span the end of one and the start of the next, and
the last item has waves without work.  Columns around the tile edges, the three
folds of y, several k blocks, and enough rows for two tiles per wave."""

import pytest

import oracle as O
from gpu_common import Guarded, check, desc_of, dev, geometry, np_of, rand_real, say, torch_gpu

pytestmark = pytest.mark.gpu

# (N_x, N_y of the shard), global N_y, k_max of y, channels
ROWS = {"even": ((5, 18), 18, 4, 3), "odd": ((5, 17), 17, 4, 3), "four": ((3, 72), 72, 32, 3),
        "k blocks": ((3, 8), 150, 72, 3), "two tiles": ((128, 6), 6, 2, 17)}
# (k_max of z, k_t): K_z K_t = 2, 14, 16, 18, 30, 64, 66, 132
COLUMNS = [(1, 1), (1, 7), (2, 4), (3, 3), (3, 5), (4, 8), (3, 11), (11, 6)]


@pytest.mark.parametrize("kz,kt", COLUMNS)
@pytest.mark.parametrize("rows", ROWS)
def test_forward_columns(rows, kz, kt):
    torch = torch_gpu()
    import paper_2607_14394_amd as D
    (nx, ny), gy, ky, c = ROWS[rows]
    nz, nt = 2 * kz + 1, 2 * kt
    g = geometry((nx, gy, nz, nt), (nx, ny, nz, nt), (0, gy - ny, 0, 0), (1, ky, kz), kt, 1, c, c)
    say(f"[axis tiles] {rows} kz={kz} kt={kt}")
    plan = D.Plan(desc_of(g), flags=D.PLAN_SPLIT_SCHEDULE)
    x = rand_real((1, c, nx, ny, nz, nt), 71)
    xhat = Guarded(torch, plan.spectral_shape(c), torch.complex64)
    plan.forward(dev(torch, x), xhat.t)
    torch.cuda.synchronize()
    check(np_of(xhat.t), O.forward(x, g), "forward")
    assert xhat.guards_intact()
    plan.close()
