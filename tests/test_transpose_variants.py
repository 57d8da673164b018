"""Transposing relayouts whose rows start anywhere: the variant in chunks that start at any element and the one whose tiles
are skewed onto the destination's lines, asked for by name at the edges of their tiles (64 .. 128 elements, a line, a chunk),
against the oracle -- the plans on the host under a bounds check, the kernels on the device with guards around the buffers."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import axe_ref as R
from oracle.axe_layout import Layout
from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W
from test_host_plans import hc, host_relayout                 # noqa: F401  (hc: the host-check library)

UINT = {1: np.uint8, 2: np.uint16, 4: np.uint32, 8: np.uint64}


def cases(eb):
    """(shape, source spec, destination spec): eS = columns, eD = rows."""
    lo = max(64 // eb, 16 // eb)                               # rows of 64 bytes are the shortest the path takes
    out = []
    for r, c in ((lo, lo), (lo + 1, 131), (129, lo + 3), (127, 257), (200, 65), (256 + 64, 128)):
        out.append(((r, c), W.row_major_spec(r, c), W.col_major_spec(r, c)))
    r, c = 130, 67 if eb < 8 else 35
    out.append(((r, c), W.spec([(r, c + 5, "m"), (c, 1, "m")], O={"m": 3}), W.spec([(r, 1, "m"), (c, r + 9, "m")], O={"m": 7})))      # pitches, offsets
    out.append(((3, r, c), W.spec([(3, r * c + 1, "m"), (r, c, "m"), (c, 1, "m")]), W.spec([(3, r * c + 11, "m"), (r, 1, "m"), (c, r, "m")])))  # batched
    out.append(((r, c), W.row_major_spec(r, c), W.spec([(r, 1, "m"), (c, r, "m")], R=[(2, -(-r * c // 128) * 128, "m")])))            # two copies, lines apart
    out.append(((r, c), W.row_major_spec(r, c), W.spec([(r, 1, "m"), (c, -r, "m")], O={"m": (c - 1) * r})))                           # destination rows backwards
    return out


def span(spec):
    e = [(n, s) for n, s, _ in spec["D"] + spec["R"]]
    return (spec["O"].get("m", 0) if spec["O"] else 0) + sum(max(0, s) * (n - 1) for n, s in e) + 1


ALL = [(eb, v, i) for eb in (1, 2, 4, 8) for v in (2, 3) if not (eb == 1 and v == 3) for i in range(10)]


@pytest.mark.parametrize("eb,variant,i", ALL)
def test_plan_on_the_host(hc, eb, variant, i):                 # noqa: F811
    shape, s, d = cases(eb)[i]
    src = np.random.default_rng(i).integers(0, 256, span(s) * eb, dtype=np.uint8).view(UINT[eb])
    for shift in (0, 3):                                       # the destination also off a line by some elements
        rng = dict(d, O={"m": (d["O"] or {}).get("m", 0) + shift})
        got, want = host_relayout(hc, Layout.from_spec(s), Layout.from_spec(rng), shape, src, span(rng), env={"AXE_TRANSPOSE_VARIANT": variant})
        assert hc.axe_hostcheck_violations() == 0 and hc.axe_hostcheck_transposes_elementwise() == 1
        assert got.tobytes() == want.tobytes()


def test_which_variant_a_copy_takes(hc):                       # noqa: F811
    """Small copies go in chunks from any element; the skew starts at 112 MiB in all, where rows do not start on lines."""
    src = np.arange(130 * 67, dtype=np.uint16)
    s, d = W.row_major_spec(130, 67), W.col_major_spec(130, 67)
    host_relayout(hc, Layout.from_spec(s), Layout.from_spec(d), (130, 67), src, src.size)
    assert hc.axe_hostcheck_transposes_elementwise() == 1 and hc.axe_hostcheck_violations() == 0
    swz = dict(W.col_major_spec(128, 64), swizzle=("m", 2, 1, 6))   # exchanges elements inside a chunk
    src = np.arange(128 * 64, dtype=np.uint16)
    got, want = host_relayout(hc, Layout.from_spec(W.row_major_spec(128, 64)), Layout.from_spec(swz), (128, 64), src, src.size,
                              env={"AXE_TRANSPOSE_VARIANT": 3})      # not taken: a swizzle
    assert got.tobytes() == want.tobytes()


@pytest.mark.gpu
@pytest.mark.parametrize("eb,variant,i", ALL)
def test_kernel_on_the_device(monkeypatch, eb, variant, i):
    monkeypatch.setenv("AXE_TRANSPOSE_VARIANT", str(variant))
    shape, s, d = cases(eb)[i]
    src = np.random.default_rng(i).integers(0, 256, span(s) * eb, dtype=np.uint8).view(UINT[eb])
    ns, nd = span(s), span(d)
    signed = {1: np.uint8, 2: np.int16, 4: np.int32, 8: np.int64}[eb]
    for lead in (0, 1, 128 // eb + 3):                         # elements before the destination: rows off a chunk, off a line
        want = np.full(nd, 0xA5, dtype=np.uint8).astype(UINT[eb])
        R.relayout_ref(Layout.from_spec(s), Layout.from_spec(d), shape, src, want)
        room = torch.from_numpy(np.full(lead + nd + 64, 0xA5, dtype=np.uint8).astype(UINT[eb]).view(signed)).cuda()
        dsrc = torch.from_numpy(np.concatenate([src, src[:64]]).view(signed)).cuda()[:ns]
        B.axe_relayout(B.Layout(s), B.Layout(d), shape, dsrc, room[lead:lead + nd])
        torch.cuda.synchronize()
        got = room.cpu().numpy().view(UINT[eb])
        assert np.array_equal(got[lead:lead + nd], want)
        assert (got[:lead] == 0xA5).all() and (got[lead + nd:] == 0xA5).all(), "written outside"
