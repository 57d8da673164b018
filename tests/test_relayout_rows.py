"""Relayouts of contiguous rows that start anywhere (padding an odd matrix, cutting a window out of one): rows around one, two
and many 16-byte chunks and one, two and several slots of 64 chunks, starts at every place of a chunk, batched and permuted
rows -- the plan on the host under a bounds check, the kernel on the device with guards, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import axe_ref as R
from oracle.axe_layout import Layout
from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W
from test_host_plans import hc, host_relayout                 # noqa: F401  (hc: the host-check library)
from test_transpose_variants import UINT, span


def cases(eb):
    lo = 256 // eb                                             # rows of 256 bytes are the shortest taken
    chunk, slot = 16 // eb, 1024 // eb
    out = []
    for n in (lo + 1, lo + chunk - 1, slot - 1, slot + 1, 2 * slot - chunk + 1, 5 * slot + 3):
        out.append(((5, n), W.row_major_spec(5, n), W.spec([(5, n + 2, "m"), (n, 1, "m")], O={"m": 1})))       # to odd pitches
        out.append(((9, n), W.spec([(9, n + 7, "m"), (n, 1, "m")], O={"m": 2}), W.row_major_spec(9, n)))        # a window, packed
    n = lo + 5
    out.append(((3, 4, n), W.row_major_spec(12, n) | {"D": [(3, 4 * n, "m"), (4, n, "m"), (n, 1, "m")]},
                W.spec([(3, n, "m"), (4, 3 * n + 1, "m"), (n, 1, "m")])))                                        # rows permuted
    out.append(((7, n), W.row_major_spec(7, n), W.spec([(7, -(n + 1), "m"), (n, 1, "m")], O={"m": 6 * (n + 1)})))  # rows backwards
    out.append(((1, 3 * slot + 1), W.spec([(1, 1, "m"), (3 * slot + 1, 1, "m")], O={"m": 3}), W.row_major_spec(1, 3 * slot + 1)))
    return out


ALL = [(eb, i) for eb in (1, 2, 4, 8) for i in range(15)]


@pytest.mark.parametrize("eb,i", ALL)
def test_plan_on_the_host(hc, eb, i):                          # noqa: F811
    shape, s, d = cases(eb)[i]
    src = np.random.default_rng(i).integers(0, 256, span(s) * eb, dtype=np.uint8).view(UINT[eb])
    for shift in range(16 // eb):
        off = dict(d, O={"m": (d["O"] or {}).get("m", 0) + shift})
        got, want = host_relayout(hc, Layout.from_spec(s), Layout.from_spec(off), shape, src, span(off))
        assert hc.axe_hostcheck_violations() == 0 and got.tobytes() == want.tobytes()
        if eb < 8 and len(shape) == 2 and shape[1] % 2:
            assert hc.axe_hostcheck_rows() == 1
        assert host_relayout(hc, Layout.from_spec(s), Layout.from_spec(off), shape, src, span(off), env={"AXE_RELAYOUT_ROWS": 0})[0].tobytes() == want.tobytes()


def test_what_stays_with_the_loop_nest(hc):                    # noqa: F811
    src = np.arange(63 * 129, dtype=np.uint16)
    plain, odd = W.row_major_spec(63, 129), W.spec([(63, 131, "m"), (129, 1, "m")])
    for s, d, shape, rows in ((plain, odd, (63, 129), 1),
                              (plain, W.spec(odd["D"], R=[(2, 63 * 131, "m")]), (63, 129), 0),                     # replicas
                              (W.row_major_spec(64, 126), W.spec([(64, 127, "m"), (126, 1, "m")]), (64, 126), 0)):  # rows of 252 bytes
        got, want = host_relayout(hc, Layout.from_spec(s), Layout.from_spec(d), shape, src[:span(s)], span(d))
        assert got.tobytes() == want.tobytes() and hc.axe_hostcheck_rows() == rows


@pytest.mark.gpu
@pytest.mark.parametrize("eb,i", ALL)
def test_kernel_on_the_device(eb, i):
    shape, s, d = cases(eb)[i]
    src = np.random.default_rng(i).integers(0, 256, span(s) * eb, dtype=np.uint8).view(UINT[eb])
    signed = {1: np.uint8, 2: np.int16, 4: np.int32, 8: np.int64}[eb]
    ns, nd = span(s), span(d)
    want = np.full(nd, 0xA5, dtype=np.uint8).astype(UINT[eb])
    R.relayout_ref(Layout.from_spec(s), Layout.from_spec(d), shape, src, want)
    for lead in (0, 1, 16 // eb - 1, 16 // eb + 1):            # elements before either buffer
        room = torch.from_numpy(np.full(lead + nd + 32, 0xA5, dtype=np.uint8).astype(UINT[eb]).view(signed)).cuda()
        dsrc = torch.from_numpy(np.concatenate([src[:lead], src]).view(signed)).cuda()[lead:lead + ns]
        B.axe_relayout(B.Layout(s), B.Layout(d), shape, dsrc, room[lead:lead + nd])
        torch.cuda.synchronize()
        got = room.cpu().numpy().view(UINT[eb])
        assert np.array_equal(got[lead:lead + nd], want)
        assert (got[:lead] == 0xA5).all() and (got[lead + nd:] == 0xA5).all(), "written outside"
