"""Dense launches of the tile family: the map from workgroups to tiles, and C stored through a descriptor at the edges of a tile."""
import ctypes as C
import os

import pytest
import torch

from paper_2601_19092_amd import binding as B
from test_tile_family import MEMBERS, check, descriptor, forced


def tile_map(grid_m, grid_n, ids):
    hc = C.CDLL(os.environ.get("AXE_TEST_HOST_LIB") or os.path.join(os.path.dirname(B.LIB_PATH), "libaxe_hostcheck.so"))
    fn = hc.axe_hostcheck_family_tile
    fn.argtypes, fn.restype = [C.c_int32] * 3 + [C.POINTER(C.c_int32)] * 2, None
    tm, tn = C.c_int32(), C.c_int32()
    out = []
    for i in ids:
        fn(i, grid_m, grid_n, C.byref(tm), C.byref(tn))
        out.append((tm.value, tn.value))
    return out


@pytest.mark.parametrize("grid_m,grid_n", [(m, n) for m in (1, 2, 3, 7, 8, 9, 15, 16, 17, 31) for n in (1, 2, 3, 8, 13, 64)] + [(1, 4099), (4099, 1), (250, 61)])
def test_every_tile_once_and_in_runs(grid_m, grid_n):
    n = grid_m * grid_n
    tiles = tile_map(grid_m, grid_n, range(n))
    assert sorted(tiles) == [(i, j) for i in range(grid_m) for j in range(grid_n)]
    # in the order of the XCDs: groups of 8 tile rows, inside them column by column
    order = [tiles[i] for x in range(8) for i in range(x, n, 8)]
    assert order == sorted(order, key=lambda t: (t[0] // 8, t[1], t[0]))


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
