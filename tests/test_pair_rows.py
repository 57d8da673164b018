"""Rows of a tile of the fused pair: what is asked for is what runs, and where nothing is, the rule's lines from both sides.  (The host layer over stand-ins of the
kernels: nothing is launched, and the addresses are made up.)"""
import ctypes as C
import os
import subprocess
import sys

import pytest

from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W

AUTO, TILES, T128, T256 = B.AXE_GROUPED_AUTO, B.AXE_GROUPED_TILES, B.AXE_GROUPED_TILES_128, B.AXE_GROUPED_TILES_256


def pair_rows(G, hidden, inter, M, hint1=AUTO, hint2=AUTO):
    hc = C.CDLL(os.environ.get("AXE_TEST_HOST_LIB") or os.path.join(os.path.dirname(B.LIB_PATH), "libaxe_hostcheck.so"))
    dt = B.AXE_F16
    d1 = B.GroupedGemmDesc(M, 2 * inter, hidden, G, B.Layout(W.row_major_spec(M, hidden)), B.Layout(W.gated_b_spec(hidden, 2 * inter, G)),
                           B.Layout(W.row_major_spec(M, inter)), M * hidden, G * 2 * inter * hidden, M * inter, dt, dt, epilogue=B.AXE_EPI_SWIGLU, kernel_hint=hint1)
    d2 = B.GroupedGemmDesc(M, hidden, inter, G, B.Layout(W.row_major_spec(M, inter)), B.Layout(W.spec([(G, hidden * inter, "m"), (inter, 1, "m"), (hidden, inter, "m")])),
                           B.Layout(W.row_major_spec(M, hidden)), M * inter, G * hidden * inter, M * hidden, dt, dt, kernel_hint=hint2)
    at = [C.c_void_p((i + 1) << 40) for i in range(7)]                                     # A, B1, H, B2, C, rows, workspace
    rc = hc.axe_gemm_grouped_pair(C.byref(d1.c), C.byref(d2.c), *at, C.c_int64(M + 1), None)
    assert rc == B.AXE_EHIP                                                                # (the stand-in answers that it has no device)
    return hc.axe_hostcheck_pair_rows()


LAYER = (128, 2048, 768)


@pytest.mark.parametrize("avg,hints,rows", [
    (180, (AUTO, AUTO), 192),
    (180, (AUTO, T128), 128), (180, (T128, AUTO), 128), (180, (T128, T128), 128), (180, (T256, T256), 256),
    (180, (TILES, TILES), 128), (180, (AUTO, TILES), 128), (180, (TILES, AUTO), 128),
    (340, (AUTO, T128), 128), (340, (TILES, TILES), 128), (340, (T128, AUTO), 128),
    (384, (TILES, TILES), 128), (385, (TILES, TILES), 256), (385, (AUTO, AUTO), 256), (385, (T128, T128), 128)])
def test_a_height_that_is_asked_for_runs(avg, hints, rows):
    assert pair_rows(*LAYER, avg * LAYER[0], *hints) == rows


@pytest.mark.parametrize("threshold,rows", [("384", 128), ("1000", 128), ("100", 256)])
def test_the_threshold_for_experiments_counts_in_a_pair(threshold, rows):
    """(read once by a process: a child)"""
    here = os.path.dirname(os.path.abspath(__file__))
    code = f"import sys; sys.path[:0] = [{here!r}, {os.path.dirname(here)!r}]; from test_pair_rows import *; print(pair_rows(*LAYER, 180 * 128))"
    out = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, AXE_GROUPED_TILE128_ROWS=threshold), capture_output=True, text=True)
    assert out.returncode == 0, out.stderr[-2000:]
    assert int(out.stdout.split()[-1]) == rows


# Rows per group on either side of each line (average or total), and tiles: columns of 256 in all groups, first and second product
@pytest.mark.parametrize("shape,M,rows", [
    (LAYER, 128 * 176, 128), (LAYER, 128 * 176 + 1, 192), (LAYER, 128 * 192, 192), (LAYER, 128 * 192 + 1, 128),
    (LAYER, 128 * 137, 128), (LAYER, 128 * 209, 128), (LAYER, 128 * 256, 128), (LAYER, 128 * 289, 128), (LAYER, 128 * 384, 128), (LAYER, 128 * 384 + 1, 256),
    ((256, 2048, 512), 256 * 184, 192), ((64, 2048, 1024), 64 * 184, 192), ((60, 2048, 1408), 60 * 184, 192),             # 448 columns and more in both
    ((224, 512, 256), 224 * 184, 192), ((223, 512, 256), 223 * 184, 128), ((56, 2048, 1024), 56 * 184, 192), ((55, 2048, 1024), 55 * 184, 128), ((64, 2048, 768), 64 * 184, 128),
    ((8, 4096, 14336), 8 * 184, 128), ((128, 512, 768), 128 * 184, 128), ((12, 4096, 3584), 12 * 184, 128), ((128, 2048, 256), 128 * 184, 128),   # few in one of them
    ((16, 4096, 2048), 16 * 256, 128), ((8, 4096, 1792), 8 * 220, 128), ((8, 2048, 1024), 8 * 240, 128), ((4, 2048, 768), 4 * 240, 128), ((1, 4096, 4096), 180, 128)])
def test_the_librarys_own_choice(shape, M, rows):
    assert pair_rows(*shape, M) == rows
