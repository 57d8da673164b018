"""Transposing relayouts with so many tiles along the source that runs of neighbours fall to one XCD: every tile is still moved once, at the counts of
tiles where a run begins (16, 32, 64), just past a window and just short of one, with a diagonal shorter and longer than a run."""
import numpy as np
import pytest
import torch

from oracle import axe_ref as R
from oracle.axe_layout import Layout
from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W
from test_host_plans import hc, host_relayout                 # noqa: F401
from test_transpose_variants import UINT

# element size, variant (2: chunks from any element, 3: skewed), tiles along the source, rows; tiles are 64 (skewed; 8-byte chunks: 64) or 128 elements wide
CASES = [(1, 2, n, 131) for n in (15, 16, 17, 31, 32, 33, 40)] + [(2, 2, 33, 400), (8, 2, 32, 70), (8, 2, 35, 9)] + \
        [(2, 3, n, 150) for n in (15, 16, 31, 33, 63, 64, 65, 130)] + [(4, 3, 64, 140), (8, 3, 66, 67)]


def sized(eb, variant, tiles, rows):
    width = (32 if eb == 8 else 64) if variant == 3 else (64 if eb == 8 else 128)
    cols = tiles * width - 3                                       # odd: rows start anywhere, the last tile is short
    return (rows, cols), W.row_major_spec(rows, cols), W.col_major_spec(rows, cols)


@pytest.mark.parametrize("eb,variant,tiles,rows", CASES)
def test_on_the_host(hc, eb, variant, tiles, rows):            # noqa: F811
    shape, s, d = sized(eb, variant, tiles, rows)
    n = shape[0] * shape[1]
    src = np.random.default_rng(tiles).integers(0, 256, n * eb, dtype=np.uint8).view(UINT[eb])
    got, want = host_relayout(hc, Layout.from_spec(s), Layout.from_spec(d), shape, src, n, env={"AXE_TRANSPOSE_VARIANT": variant})
    assert hc.axe_hostcheck_violations() == 0 and hc.axe_hostcheck_transpose_variant() == variant
    assert got.tobytes() == want.tobytes()


@pytest.mark.gpu
@pytest.mark.parametrize("eb,variant,tiles,rows", CASES)
def test_on_the_device(monkeypatch, eb, variant, tiles, rows):
    monkeypatch.setenv("AXE_TRANSPOSE_VARIANT", str(variant))
    (r, c), s, d = sized(eb, variant, tiles, rows)
    src = np.random.default_rng(tiles).integers(0, 256, r * c * eb, dtype=np.uint8).view(UINT[eb])
    signed = {1: np.uint8, 2: np.int16, 4: np.int32, 8: np.int64}[eb]
    out = torch.zeros(r * c, dtype=torch.from_numpy(src[:1].view(signed)).dtype, device="cuda")
    B.axe_relayout(B.Layout(s), B.Layout(d), (r, c), torch.from_numpy(src.view(signed)).cuda(), out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(UINT[eb]).reshape(c, r), src.reshape(r, c).T)
