"""Dense launches of the tile family: the map from workgroups to tiles, and C stored through a descriptor at the edges of a tile."""
import ctypes as C
import os

import pytest
import torch

from paper_2601_19092_amd import binding as B
from test_tile_family import MEMBERS, check, descriptor, forced


def tile_map(grid_m, grid_n, ids, member=0):
    """Tiles of these workgroups by the arguments that the planner gives a launch of grid_m x grid_n tiles (the host layer over stand-ins of the kernels: nothing
    is launched, and the addresses are made up)."""
    hc = C.CDLL(os.environ.get("AXE_TEST_HOST_LIB") or os.path.join(os.path.dirname(B.LIB_PATH), "libaxe_hostcheck.so"))
    hc.axe_gemm.argtypes = [C.POINTER(B.axe_gemm_desc_t)] + [C.c_void_p] * 4
    fn = hc.axe_hostcheck_family_tile
    fn.argtypes, fn.restype = [C.c_uint32] + [C.POINTER(C.c_int32)] * 2, None
    d = descriptor(grid_m * MEMBERS[member][0] - 1, grid_n * MEMBERS[member][1] - 1, 512)
    with forced(member):
        assert hc.axe_gemm(C.byref(d.c), 1 << 40, 1 << 41, 1 << 42, None) < 0                # (the stand-in answers that it has no device)
    assert hc.axe_hostcheck_gemm_member() == member
    tm, tn = C.c_int32(), C.c_int32()
    out = []
    for i in ids:
        fn(i, C.byref(tm), C.byref(tn))
        out.append((tm.value, tn.value))
    return out


@pytest.mark.parametrize("grid_m,grid_n", [(m, n) for m in (1, 2, 3, 7, 8, 9, 15, 16, 17, 31) for n in (1, 2, 3, 8, 13, 64)] + [(1, 4099), (4099, 1), (250, 61)])
def test_every_tile_once_and_in_runs(grid_m, grid_n):
    n = grid_m * grid_n
    tiles = tile_map(grid_m, grid_n, range(n))
    assert sorted(tiles) == [(i, j) for i in range(grid_m) for j in range(grid_n)]
    if (grid_m, grid_n) == (16, 64):                       # runs that would all start at one column of their 16 (see below)
        return
    # in the order of the XCDs: groups of 8 tile rows, inside them column by column; a run may begin further on and end with what it skipped
    key = lambda t: (t[0] // 8, t[1], t[0])
    runs = [tiles[x::8] for x in range(8)]
    starts = [r.index(min(r, key=key)) if r else 0 for r in runs]
    order = [t for r, s in zip(runs, starts) for t in r[s:] + r[:s]]
    assert not any(starts) or (n % 8 and n >= 768)
    assert order == sorted(order, key=lambda t: (t[0] // 8, t[1], t[0]))


# Grids on either side of each line, timed in runs and in blocks: four rounds and more, starts on one or two columns or a multiple of 16 columns apart
@pytest.mark.parametrize("grid_m,grid_n,blocks", [(32, 32, True), (32, 48, True), (32, 64, True), (64, 16, True), (16, 64, True), (16, 128, True), (96, 32, True),
                                                  (32, 16, False), (16, 32, False), (16, 48, False), (48, 32, False), (80, 32, False), (16, 96, False), (48, 48, False),
                                                  (32, 40, False), (40, 32, False), (31, 64, False), (32, 33, False)])
def test_which_grids_go_in_blocks(grid_m, grid_n, blocks):
    n = grid_m * grid_n
    tiles = tile_map(grid_m, grid_n, range(n), member=8)
    assert sorted(tiles) == [(i, j) for i in range(grid_m) for j in range(grid_n)]
    first = [{(i // 16, j // 16) for i, j in tiles[k:k + 256]} for k in range(0, n - n % 256, 256)]
    assert all(len(f) == 1 for f in first) == blocks
    if blocks:
        # round by round one block, neighbours after one another, and of it 8 x 4 tiles to every XCD
        order = [f.pop() for f in first]
        assert all(abs(a - c) + abs(b - d) == 1 for (a, b), (c, d) in zip(order, order[1:]))
        for x in range(8):
            i, j = zip(*tiles[x:256:8])
            assert (max(i) - min(i), max(j) - min(j)) == (7, 3)


# Grids that 8 does not divide, of three rounds and more, and neighbours that keep their starts
@pytest.mark.parametrize("grid_m,grid_n,turned", [(31, 31, True), (31, 33, True), (29, 29, True), (13, 61, True), (11, 70, True), (35, 74, True), (9, 101, True), (250, 61, True),
                                                  (13, 59, False), (15, 34, False), (7, 200, False), (28, 32, False), (15, 64, False)])
def test_starts_of_runs(grid_m, grid_n, turned):
    tiles = tile_map(grid_m, grid_n, range(grid_m * grid_n))
    assert sorted(tiles) == [(i, j) for i in range(grid_m) for j in range(grid_n)]
    key = lambda t: (t[0] // 8, t[1], t[0])
    runs = [tiles[x::8] for x in range(8)]
    assert any(r[0] != min(r, key=key) for r in runs) == turned
    if turned:
        # the 4 columns of 8 tiles that each takes first: together they lie on nearly all of the 16
        assert len({(r[0][1] + d) % 16 for r in runs for d in range(4)}) >= 14, [r[0][1] % 16 for r in runs]


def test_large_grids_divide():
    """Past the range of the factors (tiles times divisor beyond 2^31) the map divides: the same sequence."""
    gm, gn = 1003, 50021
    n = gm * gn
    q, r = n // 8, n % 8
    ids = [0, 1, 7, 8, n - 1, n - 8, n // 2, n // 3 * 2 + 1]
    for i, (tm, tn) in zip(ids, tile_map(gm, gn, ids)):
        lin = i % 8 * q + min(i % 8, r) + i // 8
        group, at = divmod(lin, 8 * gn)
        rows = min(8, gm - 8 * group)
        assert (tm, tn) == (8 * group + at % rows, at // rows)


class At:
    """An address for a scale array that nothing reads."""

    def __init__(self, dtype):
        self.dtype = dtype

    def data_ptr(self):
        return 1 << 43


@pytest.mark.parametrize("K,placed", [(512, 0), (1024, 0), (1920, 0), (2048, 1), (4096, 1)])
@pytest.mark.parametrize("scales", [None, torch.float32, torch.uint8])
def test_placed_schedule_by_k(K, placed, scales):
    """The 256 x 128 tile: E8M0 codes by K, unscaled always, fp32 scales never (both sides timed)."""
    hc = C.CDLL(os.environ.get("AXE_TEST_HOST_LIB") or os.path.join(os.path.dirname(B.LIB_PATH), "libaxe_hostcheck.so"))
    hc.axe_gemm.argtypes = [C.POINTER(B.axe_gemm_desc_t)] + [C.c_void_p] * 4
    d = descriptor(2000, 4096, K, "fp8", scales=scales and (At(scales), At(scales)))
    assert hc.axe_gemm(C.byref(d.c), 1 << 40, 1 << 41, 1 << 42, None) < 0
    assert hc.axe_hostcheck_gemm_member() == 8
    assert hc.axe_hostcheck_family_placed() == {None: 1, torch.float32: 0, torch.uint8: placed}[scales]


@pytest.mark.gpu
@pytest.mark.parametrize("K", [1920, 2048])
def test_e8m0_either_side_of_the_placed_schedule(K):
    check(8, 300, 260, K, "fp8", "bf16", "e8m0", 1, pad=1)


@pytest.mark.gpu
@pytest.mark.parametrize("member", range(len(MEMBERS)))
@pytest.mark.parametrize("dt,out,scale,rows", [("bf16", "bf16", None, 0), ("f16", "f32", None, 0), ("fp8", "bf16", "f32", 1), ("fp8", "f32", "f32", 0)])
def test_c_through_a_descriptor(member, dt, out, scale, rows):
    """Rows that exist no whole tile of, columns that end inside a fragment, a pitch of its own; nine tile rows (a second group of the map)."""
    tm, tn = MEMBERS[member][:2]
    kt = 128 if dt == "fp8" else 64
    check(member, tm + 3, tn + 12, 3 * kt, dt, out, scale, rows, pad=1)
    check(member, 8 * tm + 1, 4, 2 * kt, dt, out, scale, rows, pad=1)


@pytest.mark.gpu
@pytest.mark.parametrize("grid_m,grid_n", [(32, 32), (16, 64), (31, 31), (13, 61)])
@pytest.mark.parametrize("member", [0, 3])
def test_grids_in_blocks_and_turned_runs(member, grid_m, grid_n):
    check(member, grid_m * MEMBERS[member][0] - 3, grid_n * MEMBERS[member][1] - 4, 128, "bf16", "bf16", None, 0, pad=1)


@pytest.mark.gpu
@pytest.mark.parametrize("member", range(len(MEMBERS)))
@pytest.mark.parametrize("dt,out", [("bf16", "bf16"), ("f16", "f32")])
def test_nothing_past_the_last_row_is_written(member, dt, out):
    """One row, and one row past a whole tile: the rows that the last tile has no more of, up to two tiles of them, keep what they held."""
    tm, tn = MEMBERS[member][:2]
    tt = torch.bfloat16 if dt == "bf16" else torch.float16
    for M, N in ((1, 4), (1, tn + 12), (tm + 1, tn)):
        K, ldc = 192, N + 4
        a, b = (torch.ones((n, K), dtype=tt, device="cuda") for n in (M, N))
        held = torch.full(((M + 2 * tm) * ldc,), -7, dtype=torch.float32 if out == "f32" else tt, device="cuda")
        with forced(member):
            B.axe_gemm(descriptor(M, N, K, dt, out, ldc=ldc), a, b, held[:M * ldc])
        c = held.view(-1, ldc)
        assert (c[:M, :N] == K).all() and (c[:M, N:] == -7).all() and (c[M:] == -7).all(), (M, N)
