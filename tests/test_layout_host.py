"""Host-side checks of how calls are laid over the chip: the library's own rules, called without a GPU (functions inside
the library, by their C++ symbols)."""
import ctypes

import pytest

from paper_2601_20655_amd import binding as B
from test_abi_host import varlen_params


def packed_layout(p, nbytes):
    f = B.lib()._ZN3dit13packed_layoutEPKvmPi
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
    tiles = ctypes.c_int(-1)
    return f(ctypes.byref(p), nbytes, ctypes.byref(tiles)), tiles.value


@pytest.mark.parametrize("grids,H,nw", [
    (((1, 55, 63), (1, 40, 60), (1, 17, 18)), 3, 4),  # pieces pay, and whole tiles are faster with 4 wavefronts
    (((4, 30, 52), (1, 45, 80), (1, 30, 52)), 2, 4),
    (((1, 45, 80), (1, 40, 60)), 40, 8),
    (((1, 45, 77),), 3, 4),                           # one request: as in dit_attn_forward
])
def test_packed_call_without_room_for_pieces_takes_the_whole_tile_form(grids, H, nw):
    p = varlen_params(grids, H=H)
    room = B.dit_attn_varlen_workspace_bytes(p)
    p.flags = B.DIT_FLAG_SMALL_WORKGROUP
    whole = B.dit_attn_varlen_workspace_bytes(p)
    p.flags = 0
    assert whole <= room
    if whole < room:
        assert packed_layout(p, room) == (8, packed_layout(p, room)[1]) and packed_layout(p, room)[1] > 0
    assert packed_layout(p, whole) == (nw, 0)
    p.flags = B.DIT_FLAG_BIG_WORKGROUP
    assert packed_layout(p, whole) == (8, 0)
    p.flags = B.DIT_FLAG_SMALL_WORKGROUP
    assert packed_layout(p, room) == (4, 0)


@pytest.mark.parametrize("nb,H,Lk,split,listed", [
    (4, 40, 769, 0, False), (1, 3, 4096, 0, False), (4, 12, 4096, 0, False), (4, 40, 2048, 0, False),
    (8, 40, 2048, 0, False), (2, 40, 4096, 0, False), (16, 12, 3072, 0, True), (4, 40, 4096, 0, True), (8, 40, 4096, 2048, True),
    (2, 40, 4096, 2048, False), (1, 1, 4097, 0, True), (1, 1, 4097, 1, True), (1 << 20, 1 << 10, 4096, 0, True),
])
def test_masks_are_listed_where_the_tiles_would_read_them_too_often(nb, H, Lk, split, listed):
    f = B.lib()._ZN3dit19mask_needs_key_listEiiii
    f.restype = ctypes.c_bool
    assert f(nb, H, Lk, split) == listed


def linear_form(M, N, K, cus=256):
    """Ten times the 32-row blocks plus the 64-feature blocks of the tile a projection runs on, 0: 256 x 256 tiles."""
    f = B.lib()._ZN3dit18choose_linear_formEiiii
    f.restype = ctypes.c_int
    return f(M, N, K, cus)


def chain_layout(Lq, nb, H, nKT, D, nw=0, cus=256):
    """Wavefronts per workgroup (nw: as asked for, 0: chosen) and query tiles per workgroup of chained cross-attention."""
    f = B.lib()._ZN3dit12choose_chainEiiliiiPiS0_
    f.restype = None
    f.argtypes = 2 * [ctypes.c_int] + [ctypes.c_int64] + 3 * [ctypes.c_int] + 2 * [ctypes.POINTER(ctypes.c_int)]
    w, chain = ctypes.c_int(nw), ctypes.c_int(0)
    f(Lq, nb, H, nKT, D, cus, ctypes.byref(w), ctypes.byref(chain))
    assert w.value in (4, 8) and nw in (0, w.value)
    assert 1 <= chain.value <= min(32, (Lq + 32 * w.value - 1) // (32 * w.value) * H)  # (of one request)
    return w.value, chain.value


def test_layouts_follow_the_compute_units_of_the_device():
    """A partition of the chip has fewer compute units: 256 x 256 tiles fill it earlier, and cross-attention chains more
    query tiles per workgroup on it."""
    assert linear_form(769, 10240, 5120) == 54 and linear_form(769, 10240, 5120, cus=32) == 0
    whole, part = (chain_layout(7800, 1, 12, 3, 128, nw=8, cus=cus)[1] for cus in (256, 32))
    assert whole < part


class ChainLayout(ctypes.Structure):
    _fields_ = [("nw", ctypes.c_int), ("rows", ctypes.c_int), ("qch", ctypes.c_int)]


def call_layout(Lq, nb, H, nKT, D, two=False, cus=256, nw=0):
    """Wavefronts per workgroup, query rows per wavefront and query tiles per workgroup that a cross-attention call gets."""
    f = B.lib()._ZN3dit12layout_chainEiiliibii
    f.restype = ChainLayout
    f.argtypes = 2 * [ctypes.c_int] + [ctypes.c_int64] + 2 * [ctypes.c_int] + [ctypes.c_bool] + 2 * [ctypes.c_int]
    c = f(Lq, nb, H, nKT, D, two, cus, nw)
    return c.nw, c.rows, c.qch


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("cus", [256, 64, 32])
def test_one_round_of_query_tiles_takes_16_rows_a_wavefront(D, cus):
    """On however many compute units the device has: 64-row tiles while those are one round, then 128-row ones."""
    for nb, H in ((1, 1), (2, 3), (1, 20)):
        per = cus // (nb * H)  # tiles a head in one round
        assert call_layout(64 * per, nb, H, 5, D, cus=cus) == (4, 16, 1)
        assert call_layout(64 * per + 1, nb, H, 5, D, cus=cus) == (8, 16, 1)
        assert call_layout(128 * per, nb, H, 5, D, cus=cus, nw=4) == (8, 16, 1)
        for asked in (0, 4, 8):
            c = call_layout(128 * per + 1, nb, H, 5, D, cus=cus, nw=asked)
            assert c[1] == 32 and c[0::2] == chain_layout(128 * per + 1, nb, H, 5, D, asked, cus)
        # two softmaxes and 256-row workgroups have no such form
        assert call_layout(64, nb, H, 5, D, two=True, cus=cus)[1] == call_layout(64, nb, H, 5, D, cus=cus, nw=8)[1] == 32


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("nw", [0, 4, 8])
def test_chains_stay_inside_a_request(D, nw):
    """Chains are cut per request, whatever the batch: one query tile in all, chains longer than a head has tiles, the cap."""
    assert chain_layout(1, 1, 1, 1, D, nw)[1] == 1
    assert chain_layout(1, 500, 1, 1, D, nw)[1] == 1
    w, chain = chain_layout(300, 1, 1 << 20, 1, D, nw)  # (many heads of a few tiles each)
    assert (300 + 32 * w - 1) // (32 * w) < chain
    for nb, Lq, H in ((1, 32760, 40), (4, 32760, 40), (3, 1105, 7), (64, 77, 3)):
        for nKT in (1, 3, 13, 1000):
            chain_layout(Lq, nb, H, nKT, D, nw)


def test_chained_shapes_of_the_gpu_tests_cross_from_head_to_head():
    from test_gpu_cross_attn import CHAINS_ONE, CHAINS_TWO

    for (nb, H, tiles, keys), dims in ((CHAINS_ONE, (64, 128)), (CHAINS_TWO, (128,))):
        for D in dims:
            for nw in (4, 8):
                Lq, nKT = 32 * nw * (tiles - 1) + 11, sum((n + 63) // 64 for n in keys)
                _, chain = chain_layout(Lq, nb, H, nKT, D, nw)
                assert chain > 1 and tiles % chain != 0
                assert call_layout(Lq, nb, H, nKT, D, two=len(keys) > 1 and dims == (128,), nw=nw) == (nw, 32, chain)


def test_projection_shapes_of_the_gpu_tests_run_on_the_tiles_they_are_meant_for():
    from test_gpu_linear import STAGE_REUSE

    assert [s[0] for s in STAGE_REUSE] == [11, 21, 22, 42, 34, 44, 54]  # all that are built
    for form, stages, M, N, K in STAGE_REUSE:
        bytes_per_step = (32 * (form // 10) + 64 * (form % 10)) * 128
        room = 80 if bytes_per_step <= 26 * 1024 else 160  # two workgroups per compute unit, or one
        assert stages == min(6, room * 1024 // bytes_per_step) and K // 64 >= 2 * stages + 1
        assert linear_form(M, N, K) == form
    # and those of test_small_tiles, from one step on
    for form, M, N, K in [(11, 33, 72, 64), (11, 1, 4104, 448), (21, 2783, 144, 64), (21, 130, 3664, 704),
                          (22, 1031, 3592, 64), (22, 1031, 3592, 256), (42, 1025, 3080, 320), (34, 1250, 4104, 256),
                          (44, 3502, 1560, 64), (54, 2500, 3336, 576)]:
        assert linear_form(M, N, K) == form


def short_form(L, heads, D, table_entries, f32=False, token=False):
    """Query rows a workgroup of the kernel for short sequences (0: another kernel) and whether one launch does everything."""
    f = B.lib()._ZN3dit12choose_shortEllii
    f.restype = ctypes.c_int
    f.argtypes = 2 * [ctypes.c_int64] + 2 * [ctypes.c_int]
    g = B.lib()._ZN3dit18short_packs_itselfEliiibb
    g.restype = ctypes.c_bool
    g.argtypes = [ctypes.c_int64] + 3 * [ctypes.c_int] + 2 * [ctypes.c_bool]
    qb = f(L, heads, D, table_entries)
    return 16 * qb, qb > 0 and g(L, D, qb, table_entries, f32, token)


@pytest.mark.parametrize("L,heads,D,table,rows", [
    (1024, 4, 64, 300, 16), (1025, 1, 64, 300, 0), (1024, 5, 64, 300, 32), (1024, 8, 64, 300, 32), (1024, 9, 64, 300, 0),
    (16, 256, 64, 300, 16), (16, 257, 64, 300, 0), (17, 128, 64, 300, 16), (17, 129, 64, 300, 32), (32, 256, 64, 300, 32), (1, 1, 64, 2048, 16),
    (1, 1, 64, 2049, 0), (384, 10, 128, 468, 16), (384, 11, 128, 468, 0), (385, 1, 128, 468, 0), (1, 1, 128, 2049, 0),
])
def test_short_sequences_take_their_kernel_while_one_round_holds_them(L, heads, D, table, rows):
    assert short_form(L, heads, D, table)[0] == rows


@pytest.mark.parametrize("L,heads,D,table,f32,token,itself", [
    (256, 4, 64, 212, True, True, True), (257, 4, 64, 212, True, True, False), (512, 15, 64, 256, True, False, True), (512, 15, 64, 256, True, True, False),
    (576, 4, 64, 267, True, False, True), (768, 5, 64, 300, False, True, True), (768, 10, 64, 300, True, False, False),
    (769, 1, 64, 300, False, False, False), (64, 40, 128, 358, True, False, True), (64, 8, 128, 1387, True, False, False),
    (192, 20, 128, 402, True, False, True), (193, 8, 128, 402, True, False, False), (256, 8, 128, 694, False, False, True),
    (256, 8, 128, 1450, False, False, False), (384, 10, 128, 468, False, True, False),
])
def test_one_launch_where_it_is_faster_than_three(L, heads, D, table, f32, token, itself):
    rows, one = short_form(L, heads, D, table, f32, token)
    assert rows > 0 and one == itself


def test_short_shapes_of_the_gpu_tests_reach_every_form():
    from test_gpu_short_attn import CASES, SPLITS

    seen = set()
    for nb, grid, H, D, dtype, mode, _ in CASES:
        L = grid[0] * grid[1] * grid[2]
        table = sum(n * s // 2 for n, s in zip(grid, SPLITS[D]))
        seen.add((D, dtype) + short_form(L, nb * H, D, table, dtype == "f32", mode == "token"))
    for D, rows in ((64, 16), (64, 32), (128, 16)):
        for dtype in ("bf16", "f32"):
            assert (D, dtype, rows, True) in seen, (D, dtype, rows)
        assert any((D, dtype, rows, False) in seen for dtype in ("bf16", "f32"))
