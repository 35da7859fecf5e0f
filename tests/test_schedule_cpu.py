"""The kernels that plans take (dtst_desc_schedule, host only): the parity
tests' geometries reach the kernels they are meant for."""

import pytest

D = pytest.importorskip("paper_2607_14394_amd", reason="libdtst.so not built")

from test_gpu_t_chunks import ROW_BLOCKS, SHORT_ROWS  # noqa: E402
from test_gpu_z_first import CASES, FUSED, T_FIRST, fused_case  # noqa: E402


def schedule(case, flags=0):
    return D.dtst_desc_schedule(D.make_desc(*case), flags)


@pytest.mark.parametrize("name", list(CASES))
def test_z_first_cases(name):
    s, split = schedule(CASES[name]), schedule(CASES[name], D.PLAN_SPLIT_SCHEDULE)
    assert split.forward == D.ROWS_Z_FIRST
    if name.startswith("zy_"):
        assert s.forward == D.ROWS_Z_FIRST_Y and not s.z_mirrored
        assert (s.y_parts > 1) == ("parts" in name)
        return
    assert s.forward >= D.ROWS_Z_FIRST and s.inverse >= D.ROWS_Z_FIRST and split.inverse == D.ROWS_Z_FIRST
    if name.startswith("rows_"):
        assert s.forward == s.inverse == D.ROWS_Z_FIRST and not s.z_mirrored


@pytest.mark.parametrize("name", list(T_FIRST))
def test_t_first_cases(name):
    s = schedule(T_FIRST[name])
    n_t = T_FIRST[name][1][3]
    assert s.forward == D.ROWS_T_FIRST and s.t_folded == (n_t == 32)
    assert (s.inverse == D.ROWS_T_FIRST) == (n_t == 32)


def test_z_first_cases_cover_the_unfolded_fused_forward():
    """Each (t groups, K_t tiles, y folded) of fwd_zty_kernel without mirrored rows."""
    seen = set()
    for c in CASES.values():
        s = schedule(c)
        if s.forward == D.ROWS_Z_FIRST_Y and not s.z_mirrored:
            ng, nl, _, _, kt = c[:5]
            seen.add((1 if nl[3] <= 16 else 2, 1 if kt <= 8 else 2, nl[1] == ng[1] and ng[1] % 2 == 0))
    assert seen == {(1, 1, False), (1, 1, True), (2, 1, False), (2, 1, True), (2, 2, False), (2, 2, True)}


def test_fused_cases_cover_the_mirrored_fused_forward():
    """Each (t groups, K_t tiles, y folded, whole units, z classes of the t-first rows) with mirrored rows, and with
    one t group and several classes one unit and more."""
    seen = set()
    for case in FUSED:
        c = fused_case(case)
        s = schedule(c)
        assert s.forward == D.ROWS_Z_FIRST_Y and s.z_mirrored, case
        ng, nl, _, _, kt = c[:5]
        seen.add((1 if nl[3] <= 16 else 2, 1 if kt <= 8 else 2, nl[1] == ng[1] and ng[1] % 2 == 0, ng[2] % 32 == 0,
                  s.z_classes > 1))
        if nl[3] <= 16 and s.z_classes > 1:
            seen.add(("one unit" if ng[2] <= 32 else "units", nl[1] % 2 == 0, ng[2] % 32 == 0))
    flags = [(y, w, c) for y in (False, True) for w in (False, True) for c in (False, True)]
    assert seen == ({(th, mk) + f for th, mk in ((1, 1), (2, 1), (2, 2)) for f in flags}
                    | {(u, y, w) for u in ("one unit", "units") for y in (False, True) for w in (False, True)})


def test_t_first_forward_is_fused_at_whole_quads_of_t():
    """N_t % 4 == 0: y in the t-first forward's launch; otherwise launches of its own (the inverse stays fused)."""
    for nt, way in ((28, D.ROWS_T_FIRST_Y), (30, D.ROWS_T_FIRST)):
        n = (52, 76, 38, nt)
        s = schedule((n, (26, 19) + n[2:], (0, 0, 0, 0), (22, 12, 16), 4, 3, 8, 8))
        assert s.forward == way
        assert s.inverse in (D.ROWS_T_FIRST_Y, D.ROWS_Z_FIRST_Y)


def test_z_first_forward_with_empty_y_slots():
    """Over a quarter of the last group's 16 y slots empty: y in launches of its own, unless the plan has no W1
    (N_t = 32, fused t-first kernels) or the rows form shorter chains (four z classes)."""
    for n, k, way in (((18, 18, 187, 28), (5, 8, 10), D.ROWS_Z_FIRST), ((18, 24, 187, 28), (5, 8, 10), D.ROWS_Z_FIRST_Y),
                      ((16, 16, 148, 26), (6, 7, 4), D.ROWS_Z_FIRST_Y)):
        assert schedule((n, n, (0, 0, 0, 0), k, 3, 1, 4, 4)).forward == way, n


@pytest.mark.parametrize("case", ROW_BLOCKS + SHORT_ROWS, ids=str)
def test_row_block_cases(case):
    ng, kz, kt, ci, co, shard = case
    off, nz = shard if shard else (0, ng[2])
    s = schedule((ng, (ng[0], ng[1], nz, ng[3]), (0, 0, off, 0), (1, 1, kz), kt, 2, ci, co))
    assert s.block == (D.BLOCK_ROW_TASKS if case in ROW_BLOCKS else D.BLOCK_CHUNKS)


# (n, k_max z, k_t, C_in, C_out), fused: blocks whose folded z image leaves the chunked kernel too little LDS
LONG_BLOCKS = [((2, 3, 288, 28), 8, 15, 20, 20, True), ((2, 2, 388, 28), 5, 13, 20, 20, True),
               ((2, 2, 386, 28), 10, 11, 16, 16, True), ((2, 2, 480, 28), 8, 9, 32, 32, True),
               ((2, 2, 402, 28), 7, 9, 28, 28, False), ((2, 2, 347, 20), 11, 11, 16, 16, False)]


@pytest.mark.parametrize("case", LONG_BLOCKS, ids=str)
def test_long_blocks_keep_the_fused_kernel_unfolded(case):
    n, kz, kt, ci, co, fused = case
    s = schedule((n, n, (0, 0, 0, 0), (1, 1, kz), kt, 2, ci, co))
    assert not s.t_folded
    assert (s.block, s.block_t_folded) == ((D.BLOCK_CHUNKS, 0) if fused else (D.BLOCK_SEPARATE, 1))


def test_schedule_flags_and_errors():
    c = ((12, 10, 8, 8), (4, 10, 8, 8), (4, 0, 0, 0), (3, 2, 2), 3, 1, 2, 3)
    assert schedule(c).forward in (D.ROWS_T_FIRST_Y, D.ROWS_Z_FIRST_Y)
    assert schedule(c, D.PLAN_SPLIT_SCHEDULE).forward in (D.ROWS_T_FIRST, D.ROWS_Z_FIRST)
    assert schedule(c, D.PLAN_UNFUSED_BLOCK).block == D.BLOCK_SEPARATE
    with pytest.raises(D.DtstError):
        schedule(c, 4)
    with pytest.raises(D.DtstError):
        schedule(c[:4] + (17,) + c[5:])
