"""The attention's plan on the host: over units, query rows, table widths and workspaces from the least one on, every
segment's page ids fit the kernels' LDS table, the scratch in use fits the workspace, and the least workspace stays at
one partial result per prefix chunk (and, for bf16, two lists of the chunks)."""
import ctypes as C

import pytest

from paper_2608_04962_amd import _lib

SEG_TILES, BLOCKS, TILE = 1024, 256, 64        # tiles whose page ids the LDS table holds; blocks; keys per tile


class Plan(C.Structure):
    _fields_ = [("R", C.c_int), ("Rpad", C.c_int), ("row_groups", C.c_int), ("group_rows", C.c_int),
                ("whole", C.c_bool), ("min_tiles", C.c_int), ("unit_cost", C.c_int), ("n_ranges", C.c_longlong),
                ("part_o_bytes", C.c_size_t), ("part_ml_bytes", C.c_size_t), ("work_bytes", C.c_size_t),
                ("min_bytes", C.c_size_t), ("full_bytes", C.c_size_t), ("each", C.c_bool),
                ("pairs", C.c_bool), ("by_unit", C.c_bool)]


def _plan(d, avail):
    f = getattr(_lib.lib(), "_ZN2sr9attn_planERK12sr_attn_descm")
    f.restype, f.argtypes = Plan, [C.POINTER(_lib.AttnDesc), C.c_size_t]
    return f(C.byref(d), avail)


def _up(x):
    return -(-x // 256) * 256


def _least(d, p):
    units = d.B * d.Hkv * p.row_groups
    cp = 32 if units < 64 else 128 if units < 512 else 256
    nch = max(1, -(-d.max_blocks // cp))
    rows = d.B * d.Hkv * nch * p.Rpad
    parts = _up(rows * d.D * 4) + _up(rows * 8) if nch > 1 else 0
    return parts + (_up((3 + 2 * units * nch) * 4) if d.dtype == _lib.SR_BF16 else 0), nch


def _check(d, avail):
    p = _plan(d, avail)
    units = d.B * d.Hkv * p.row_groups
    most = -(-d.max_blocks * 16 // TILE) + -(-d.T // TILE)
    total = units * (most + p.unit_cost)
    # tiles of a range, as the kernels cut the longest contexts that the table can hold
    grid = min(p.n_ranges, BLOCKS)
    ranges = min(p.n_ranges, grid * -(-total // grid // SEG_TILES) if total > grid * SEG_TILES else grid)
    length = max(p.min_tiles, -(-total // ranges))
    assert p.each == (p.whole and units <= BLOCKS)
    if p.each or p.pairs:                      # a range for each unit, or for two, of any length
        assert p.n_ranges == (units if p.each else BLOCKS) and (p.each or units <= 2 * BLOCKS and d.B <= 2 * BLOCKS)
        length = 1
    assert length <= SEG_TILES
    assert (most if p.whole else min(most, length)) <= SEG_TILES, "a segment's page ids overrun the LDS table"
    used = p.part_o_bytes + p.part_ml_bytes + p.work_bytes
    assert used <= avail, (used, avail)
    if not p.whole:
        n = -(-total // length)                # ranges; the last partial result that any of them may write
        assert n <= p.n_ranges
        last = n + units - 1 if p.by_unit else 2 * n
        assert last * p.group_rows * d.D * 4 <= p.part_o_bytes and last * p.group_rows * 8 <= p.part_ml_bytes
        assert p.work_bytes >= (1 + d.B) * 8
    return p


@pytest.mark.parametrize("dtype", [_lib.SR_F32, _lib.SR_BF16])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,G", [(1, 1), (8, 4), (8, 7), (13, 5), (32, 7), (32, 8), (65, 4), (64, 5), (128, 16)])
def test_plan_over_workspaces(dtype, D, T, G):
    for B, Hkv in ((1, 1), (1, 4), (3, 1), (8, 8), (63, 1), (64, 8), (67, 8), (128, 4), (256, 8), (1024, 8), (65535, 1)):
        for max_blocks in (1, 10, 32, 33, 64, 129, 256, 257, 512, 1025, 4096, 7680, 8192, 15872, 65536):
            d = _lib.AttnDesc(B, T, Hkv * G, Hkv, D, 16, max_blocks, 1 << 20, dtype, 0.1)
            full = _plan(d, C.c_size_t(-1).value)
            least, nch = _least(d, full)
            assert full.min_bytes == least and full.full_bytes == _lib.lib().sr_tree_verify_attn_workspace(C.byref(d))
            for avail in sorted({least, least + 256, (least + full.full_bytes) // 2, full.full_bytes - 1, full.full_bytes}):
                if avail >= least:
                    p = _check(d, avail)
                    assert p.min_bytes == least, "a workspace that was enough is refused"
                    if nch > 3:                # a long prefix is still cut, or there are units for half the blocks
                        assert not p.whole or B * Hkv * p.row_groups >= BLOCKS // 2


def test_ranges_past_the_table_come_in_whole_rounds():
    """More tiles than 256 blocks' tables hold: every block gets the same number of ranges."""
    for dtype in (_lib.SR_F32, _lib.SR_BF16):
        for B, mb in ((64, 2048), (64, 2100), (67, 7680), (1024, 1024), (300, 4096)):
            d = _lib.AttnDesc(B, 8, 8, 8, 64, 16, mb, 1 << 20, dtype, 0.1)
            p = _check(d, C.c_size_t(-1).value)
            assert p.n_ranges > BLOCKS and p.n_ranges % BLOCKS == 0, p.n_ranges


def test_few_units_of_any_length():
    """One to five units: 64 pieces each, more of long ones and where their page ids would not fit."""
    for dtype in (_lib.SR_F32, _lib.SR_BF16):
        for units in range(1, 6):
            for mb in (200, 2000, 20000, 1 << 20, 1 << 22, 1 << 25):
                d = _lib.AttnDesc(1, 8, 8 * units, units, 64, 16, mb, 1 << 20, dtype, 0.1)
                p = _check(d, C.c_size_t(-1).value)
                if mb <= 2000:
                    assert p.n_ranges <= min(64 * units, BLOCKS)
                assert p.n_ranges <= BLOCKS or p.n_ranges % BLOCKS == 0
                least, _ = _least(d, p)
                _check(d, least)


def test_units_left_whole():
    """Short units are left whole, the longer the more blocks they fill, and need no partial results; a unit past the
    line is cut."""
    for dtype, B, Hkv, tiles in ((_lib.SR_BF16, 64, 4, 24), (_lib.SR_BF16, 32, 4, 14), (_lib.SR_BF16, 1, 1, 4),
                                 (_lib.SR_BF16, 65, 4, 26), (_lib.SR_BF16, 128, 4, 26), (_lib.SR_BF16, 129, 4, 7),
                                 (_lib.SR_BF16, 512, 8, 7), (_lib.SR_F32, 64, 4, 6),
                                 (_lib.SR_F32, 1, 4, 4), (_lib.SR_F32, 128, 4, 4)):
        for more in (0, 1):
            d = _lib.AttnDesc(B, 8, 7 * Hkv, Hkv, 128, 16, 4 * (tiles - 1 + more), 1 << 20, dtype, 0.1)
            p = _check(d, C.c_size_t(-1).value)
            assert p.whole == (more == 0) and (p.part_o_bytes == 0) == p.whole, (dtype, B, Hkv, tiles, more)


def test_partial_results_follow_the_rows():
    """Few query rows per KV head ask for the scratch of these rows, not of a full row group."""
    for dtype in (_lib.SR_F32, _lib.SR_BF16):
        for T, G in ((1, 1), (8, 4), (8, 7), (32, 7)):
            d = _lib.AttnDesc(4, T, 4 * G, 4, 128, 16, 1024, 1 << 20, dtype, 0.1)
            p = _check(d, C.c_size_t(-1).value)
            assert p.group_rows == -(-T * G // 32) * 32
            assert p.part_o_bytes <= (256 + 4 * 4) * p.group_rows * 128 * 4


def test_noalloc_takes_what_fits_its_array_with_segments_in_the_table():
    """Requests whose least scratch fits the library's own array while their full one does not."""
    cap = 256 << 20
    for B, T, Hkv, G, D, mb, dtype in ((64, 8, 8, 4, 64, 15872, _lib.SR_F32), (67, 8, 8, 4, 128, 7680, _lib.SR_F32),
                                       (64, 32, 8, 1, 64, 15000, _lib.SR_BF16)):
        d = _lib.AttnDesc(B, T, Hkv * G, Hkv, D, 16, mb, 1 << 20, dtype, 0.1)
        p = _plan(d, C.c_size_t(-1).value)
        assert p.min_bytes <= cap
        _check(d, cap)
