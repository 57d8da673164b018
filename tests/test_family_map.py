"""Dense launches of the tile family: which way a grid of tiles goes to the XCDs, and which launches have their reads and loads placed, as the planner has it."""
import ctypes as C
import os

import pytest
import torch

from paper_2601_19092_amd import binding as B
from test_tile_family import MEMBERS, check, descriptor, forced


def planned_map(grid_m, grid_n, ids, member=0):
    """Tiles of these workgroups by the arguments that the planner gives a launch of grid_m x grid_n tiles (the host layer over stand-ins of the kernels: nothing
    is launched, and the addresses are made up)."""
    hc = C.CDLL(os.environ.get("AXE_TEST_HOST_LIB") or os.path.join(os.path.dirname(B.LIB_PATH), "libaxe_hostcheck.so"))
    hc.axe_gemm.argtypes = [C.POINTER(B.axe_gemm_desc_t)] + [C.c_void_p] * 4
    fn = hc.axe_hostcheck_planned_tile
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


# Grids on either side of each line, timed in runs and in blocks: four rounds and more, starts on one or two columns or a multiple of 16 columns apart
@pytest.mark.parametrize("grid_m,grid_n,blocks", [(32, 32, True), (32, 48, True), (32, 64, True), (64, 16, True), (16, 64, True), (16, 128, True), (96, 32, True),
                                                  (32, 16, False), (16, 32, False), (16, 48, False), (48, 32, False), (80, 32, False), (16, 96, False), (48, 48, False),
                                                  (32, 40, False), (40, 32, False), (31, 64, False), (32, 33, False)])
def test_which_grids_go_in_blocks(grid_m, grid_n, blocks):
    n = grid_m * grid_n
    tiles = planned_map(grid_m, grid_n, range(n), member=8)
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
    tiles = planned_map(grid_m, grid_n, range(grid_m * grid_n))
    assert sorted(tiles) == [(i, j) for i in range(grid_m) for j in range(grid_n)]
    key = lambda t: (t[0] // 8, t[1], t[0])
    runs = [tiles[x::8] for x in range(8)]
    assert any(r[0] != min(r, key=key) for r in runs) == turned
    if turned:
        # the 4 columns of 8 tiles that each takes first: together they lie on nearly all of the 16
        assert len({(r[0][1] + d) % 16 for r in runs for d in range(4)}) >= 14, [r[0][1] % 16 for r in runs]


def panels(tiles, tm, tn):
    """Rows of A and B that the XCDs read between them, one round of tiles: each panel once for every XCD that has a tile of it."""
    return sum(len({i for i, _ in tiles[x::8]}) * tm + len({j for _, j in tiles[x::8]}) * tn for x in range(8))


def in_turn(grid_m, grid_n):
    return [(8 * (i // (8 * grid_n)) + i % (8 * grid_n) % min(8, grid_m - i // (8 * grid_n) * 8), i % (8 * grid_n) // min(8, grid_m - i // (8 * grid_n) * 8)) for i in range(grid_m * grid_n)]


def in_runs(grid_m, grid_n):
    seq, n = in_turn(grid_m, grid_n), grid_m * grid_n
    return [seq[i % 8 * (n // 8) + min(i % 8, n % 8) + i // 8] for i in range(n)]


@pytest.mark.parametrize("member", range(len(MEMBERS)))
def test_one_round_goes_in_turn_unless_that_reads_more(member):
    """All grids of up to 256 tiles that 8 does not divide, of every height that has a second group of tile rows, against a count of the panels."""
    tm, tn = MEMBERS[member][:2]
    seen = set()
    for grid_m in [*range(9, 34), 52, 53, 54, 81, 116, 127, 255]:
        for grid_n in range(1, 256 // grid_m + 1):
            if grid_m * grid_n % 8 == 0 or (grid_m + grid_n + member) % 3:
                continue
            runs, turns = in_runs(grid_m, grid_n), in_turn(grid_m, grid_n)
            want = turns if 20 * panels(turns, tm, tn) < 23 * panels(runs, tm, tn) else runs
            assert planned_map(grid_m, grid_n, range(grid_m * grid_n), member) == want, (grid_m, grid_n)
            seen.add(want is turns)
    assert seen == {True, False}


# timed on either side: the slowest in runs, and others that stay in runs (two rounds; up to 8 tile rows; many fewer panels)
@pytest.mark.parametrize("member,grid_m,grid_n,turn", [(6, 53, 4, True), (6, 26, 6, True), (4, 12, 15, True), (3, 81, 3, True), (5, 239, 1, True), (4, 9, 18, True),
                                                       (8, 10, 30, False), (0, 1, 166, False), (4, 7, 30, False), (1, 14, 11, False)])
def test_which_grids_go_in_turn(member, grid_m, grid_n, turn):
    assert (planned_map(grid_m, grid_n, range(grid_m * grid_n), member) == in_turn(grid_m, grid_n)) == turn


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
@pytest.mark.parametrize("grid_m,grid_n", [(32, 32), (16, 64), (31, 31), (13, 61)])
@pytest.mark.parametrize("member", [0, 3])
def test_grids_in_blocks_and_turned_runs(member, grid_m, grid_n):
    check(member, grid_m * MEMBERS[member][0] - 3, grid_n * MEMBERS[member][1] - 4, 128, "bf16", "bf16", None, 0, pad=1)


@pytest.mark.gpu
@pytest.mark.parametrize("member,grid_m,grid_n", [(6, 26, 6), (4, 12, 15), (3, 81, 3), (0, 9, 1)])
@pytest.mark.parametrize("dt,out", [("bf16", "bf16"), ("f16", "f32")])
def test_grids_in_turn(member, grid_m, grid_n, dt, out):
    check(member, grid_m * MEMBERS[member][0] - 3, grid_n * MEMBERS[member][1] - 4, 136, dt, out, None, 0, pad=1)
