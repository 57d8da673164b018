"""Which kernel a relayout goes to, and in how many workgroups, for copies too large to be made on the host: the plan alone is
made (the stand-ins of libaxe_hostcheck.so move nothing)."""
import ctypes as C

import pytest

from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W
from test_host_plans import hc                                 # noqa: F401

LIMIT = 1 << 32                                                # HIP refuses a launch of that many threads


@pytest.fixture
def plan(hc):                                                  # noqa: F811
    """(rc, variant of the transposing kernel or None, "rows" / "tiles" / "nest", workgroups) of a relayout."""
    hc.axe_hostcheck_workgroups.restype = C.c_int64

    def run(shape, s, d, eb, src=1 << 12, dst=1 << 45):
        ls, ld = B.Layout(s), B.Layout(d)
        hc.axe_hostcheck_set_buffers(1 << 44, 1 << 44)
        hc.axe_hostcheck_plan_only(1)
        try:
            rc = hc.axe_relayout(C.byref(ls.c), C.byref(ld.c), len(shape), (C.c_int64 * len(shape))(*shape), eb, 0, src, (1 << 44) // eb,
                                 dst, (1 << 44) // eb, None)
        finally:
            hc.axe_hostcheck_plan_only(0)
        if hc.axe_hostcheck_transposes():
            return rc, hc.axe_hostcheck_transpose_variant(), "tiles", hc.axe_hostcheck_workgroups()
        return rc, None, "rows" if hc.axe_hostcheck_rows() else "nest", hc.axe_hostcheck_workgroups()
    return run


def batched(b, r, c, src_pad=0, dst_pad=0):
    """b matrices of r x c from row-major (rows src_pad apart) to column-major."""
    return ((b, r, c), W.spec([(b, r * (c + src_pad), "m"), (r, c + src_pad, "m"), (c, 1, "m")]),
            W.spec([(b, (r + dst_pad) * c, "m"), (r, 1, "m"), (c, r + dst_pad, "m")]))


@pytest.mark.parametrize("eb", [1, 2, 4, 8])
@pytest.mark.parametrize("b", [1 << 18, (1 << 21) - 1, 1 << 21, (1 << 23) + 5, (1 << 24) - 1])
def test_many_small_matrices_fit_one_launch(plan, b, eb):
    """Up to 2^24 - 1 matrices of one tile each: no grid padding may take the launch past what HIP accepts."""
    n = max(64 // eb, 8) + 1
    for shape, s, d in (batched(b, 64, n, src_pad=1), batched(b, 64, n)):
        if n > 64:
            shape, s, d = batched(b // 2, 64, n)               # (two tiles of 64)
        rc, _, how, wgs = plan(shape, s, d, eb)
        assert rc == B.AXE_OK and how == "tiles" and wgs * 256 < LIMIT


def test_more_than_one_launch_of_tiles_goes_to_the_loop_nest(plan):
    rc, _, how, _ = plan(*batched(1 << 24, 8, 9), 8)           # 2^24 workgroups of 256
    assert rc == B.AXE_OK and how == "nest"
    assert plan(*batched(1 << 24, 33, 33), 2)[0] == B.AXE_EUNSUPPORTED   # ... nor does that hold 2^24 x 1089 elements


@pytest.mark.parametrize("c", [100, 129, 500, 1000, 1031, 2047, 3298, 7001, 8193])
def test_padding_adds_few_workgroups(plan, c):
    """The grid is padded along the source only where the empty workgroups are few: an eighth, in a large matrix a quarter."""
    for b, r in ((1, 4001), (3, 400), (40, 129), (1, 7955)):
        rc, v, how, wgs = plan(*batched(b, r, c), 2)
        assert rc == B.AXE_OK and how == "tiles"
        if v == 2:
            tiles = b * -(-r // 128) * -(-c // 128)
            large = r >= 1000 and 4 * b * r * c >= 48 << 20
            assert tiles <= wgs and (4 * wgs <= 5 * tiles if large else 8 * wgs <= 9 * tiles)
            if (r, c) == (7955, 3298):
                assert wgs == 63 * 32


def padded_rows(rows, n, pad=1):
    return (rows, n), W.row_major_spec(rows, n), W.spec([(rows, n + pad, "m"), (n, 1, "m")])


@pytest.mark.parametrize("rows", [1 << 20, (1 << 28) - 16, (1 << 28) - 12, 1 << 28, (1 << 28) + (1 << 20)])
def test_rows_beyond_one_launch_go_to_the_loop_nest(plan, rows):
    """A slot per row: 2^28 slots are 2^24 workgroups.  What holds more stays with the loop nest, which serves it."""
    rc, _, how, wgs = plan(*padded_rows(rows, 33), 8)          # (264 bytes, in units of 8; a multiple of 4 rows: the nest unrolls them)
    assert rc == B.AXE_OK and (how == "nest" or rows <= 16 * ((1 << 24) - 1) and wgs * 256 < LIMIT)
    rc, _, how, wgs = plan(*padded_rows(1 << 20, 4095), 1)     # up to 257 chunks, five slots a row
    assert rc == B.AXE_OK and how == "rows" and wgs == 5 << 16


CHUNKS, ELEMENTS, ANY_START, SKEWED = 0, 1, 2, 3


@pytest.mark.parametrize("eb,b,r,c,variant", [
    # single bytes: chunks from any element at every size
    (1, 100000, 65, 65, ANY_START), (1, 1000, 65, 65, ANY_START), (1, 1, 8191, 8193, ANY_START),
    # matrices inside one tile of 64: element by element
    (2, 1000, 33, 33, ELEMENTS), (2, 100000, 33, 33, ELEMENTS), (2, 20000, 64, 33, ELEMENTS), (4, 1000, 33, 33, ELEMENTS), (4, 200000, 16, 17, ELEMENTS),
    # more than one: the tiles of 128 are fewer
    (2, 60000, 66, 66, ANY_START), (2, 1000, 257, 100, ANY_START), (2, 1, 700000, 33, ANY_START), (2, 16, 4097, 77, ANY_START), (2, 5000, 127, 129, ELEMENTS),
    (4, 1, 100000, 33, ELEMENTS), (4, 300, 200, 65, ANY_START), (4, 2, 531, 700, ELEMENTS), (4, 1, 4785, 1217, ANY_START), (4, 1, 9253, 1016, ELEMENTS),
    # out to memory: skewed where that does not take many more tiles
    (2, 1, 8191, 8193, SKEWED), (2, 2000, 200, 201, SKEWED), (2, 4000, 33, 1001, ANY_START), (4, 4000, 1001, 33, SKEWED), (4, 4000, 33, 1001, ELEMENTS),
    (4, 1, 17, 3000001, ELEMENTS), (4, 1, 3000001, 17, SKEWED), (4, 12000, 130, 130, ELEMENTS), (4, 2671, 161, 177, SKEWED), (8, 200000, 9, 8, SKEWED), (8, 30000, 50, 41, ELEMENTS),
    # aligned chunks, rows off the lines: a matrix inside one tile shares none
    (2, 1, 8184, 8200, SKEWED), (2, 2000, 200, 200, SKEWED), (2, 30000, 72, 72, CHUNKS), (2, 100000, 40, 40, CHUNKS), (4, 100000, 40, 40, SKEWED),
    (4, 20000, 72, 72, CHUNKS), (8, 100000, 24, 24, SKEWED), (8, 30000, 56, 56, CHUNKS)])
def test_variant_of_a_transpose(plan, eb, b, r, c, variant):
    """The variant that was the fastest, or level with it, when all that serve the copy were timed."""
    rc, got, how, _ = plan(*batched(b, r, c), eb)
    assert rc == B.AXE_OK and how == "tiles" and got == variant


@pytest.mark.parametrize("rows,n,eb,pad,how", [
    # (row bytes, unit, rows the nest unrolls by) 16 bytes per lane and more: the nest
    (60000, 33, 8, 1, "nest"), (60000, 66, 4, 1, "nest"), (400000, 66, 4, 2, "nest"), (60000, 375, 8, 1, "nest"), (60002, 375, 8, 1, "nest"),
    # 8 bytes: from 704 on
    (60001, 65, 8, 1, "nest"), (60001, 97, 8, 1, "rows"), (60002, 129, 4, 1, "nest"), (60002, 193, 4, 1, "rows"), (60000, 260, 2, 1, "nest"),
    (60000, 385, 2, 1, "rows"),
    # 4 bytes: from 448 on
    (60001, 65, 4, 1, "nest"), (60001, 129, 4, 1, "rows"), (20002, 161, 2, 1, "nest"), (20002, 225, 2, 1, "rows"), (60000, 257, 1, 1, "nest"),
    (60000, 515, 1, 1, "rows"),
    # 2 bytes and single ones
    (20001, 129, 2, 1, "rows"), (60002, 257, 1, 1, "nest"), (60002, 321, 1, 1, "rows"), (20001, 257, 1, 1, "rows"), (3001, 515, 1, 1, "nest"),
    (8191, 8191, 2, 1, "rows"), (4097, 4095, 4, 1, "rows"), (9, 257, 1, 1, "rows")])
def test_rows_or_loop_nest(plan, rows, n, eb, pad, how):
    """The kernel that was the faster one, or level with the other, when both were timed."""
    rc, _, got, _ = plan(*padded_rows(rows, n, pad), eb)
    assert rc == B.AXE_OK and got == how


def test_permuted_rows_of_a_few_hundred_bytes_stay_with_the_nest(plan):
    b, h, n = 4000, 16, 132                                    # (token, head, d) -> (head, token, d)
    s, d = W.spec([(b, h * n, "m"), (h, n, "m"), (n, 1, "m")]), W.spec([(b, n, "m"), (h, b * n, "m"), (n, 1, "m")])
    assert plan((b, h, n), s, d, 2)[0::2] == (B.AXE_OK, "nest")
