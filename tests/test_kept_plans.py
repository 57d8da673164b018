"""axe_relayout and axe_layout_eval keep the plan of a thread's last call: calls that differ in one word of a layout, in the
shape, in the buffers' alignment or in a knob get a plan of their own, and the checks of pointers and counts run on every call."""
import ctypes as C
import threading

import numpy as np

from oracle import axe_ref as R
from oracle.axe_layout import Layout
from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W
from test_host_plans import hc                                 # noqa: F401


def call(hc, s, d, shape, src, dst, s_elems=None, d_elems=None):   # noqa: F811
    ls, ld = B.Layout(s), B.Layout(d)
    hc.axe_hostcheck_set_buffers(src.nbytes, dst.nbytes)
    return hc.axe_relayout(C.byref(ls.c), C.byref(ld.c), len(shape), (C.c_int64 * len(shape))(*shape), src.itemsize, 0, src.ctypes.data,
                           src.size if s_elems is None else s_elems, dst.ctypes.data, dst.size if d_elems is None else d_elems, None)


def right(hc, s, d, shape, src, dst):                          # noqa: F811
    want = dst.copy()
    R.relayout_ref(Layout.from_spec(s), Layout.from_spec(d), shape, src, want)
    assert call(hc, s, d, shape, src, dst) == B.AXE_OK and hc.axe_hostcheck_violations() == 0
    assert dst.tobytes() == want.tobytes()


def test_relayout_plans(hc, monkeypatch):                      # noqa: F811
    src = np.arange(40000, dtype=np.uint16)
    room = np.zeros(40000 + 64, dtype=np.uint16)
    base = room[(-room.ctypes.data % 128) // 2:][:40000]       # on a line
    s, d = W.row_major_spec(128, 256), W.col_major_spec(128, 256)
    steps = [(s, d, (128, 256)), (s, d, (128, 256)), (s, W.row_major_spec(128, 256), (128, 256)), (s, d, (256, 128)),
             (s, dict(d, O={"m": 8}), (128, 256)), (s, dict(d, O={"m": 3}), (128, 256)), (s, d, (32768,)),
             (s, W.spec([(128, 1, "m"), (256, 130, "m")]), (128, 256)), (W.spec([(128, 260, "m"), (256, 1, "m")]), d, (128, 256)),
             (s, W.blocked_swizzled_spec(128, 256), (128, 256)), (s, W.blocked_swizzled_spec(128, 256, swizzle=False), (128, 256))]
    for a, b, shape in steps:
        for lead in (0, 1, 8, 0):                              # other alignments of the destination
            if shape != (256, 128):
                right(hc, a, b, shape, src, base[lead:])
    right(hc, s, d, (128, 256), src, base)
    monkeypatch.setenv("AXE_TRANSPOSE_VARIANT", "1")           # a knob is heeded by the very next call
    right(hc, s, d, (128, 256), src, base)
    assert hc.axe_hostcheck_transposes_elementwise() == 1
    monkeypatch.delenv("AXE_TRANSPOSE_VARIANT")
    right(hc, s, d, (128, 256), src, base)
    assert hc.axe_hostcheck_transposes_elementwise() == 0
    # checks of the buffers on a kept plan
    assert call(hc, s, d, (128, 256), src, src) == B.AXE_EINVAL                      # overlap
    assert call(hc, s, d, (128, 256), src, base, d_elems=128 * 256 - 1) == B.AXE_ERANGE
    assert call(hc, s, d, (128, 256), src, base, s_elems=128 * 256 - 1) == B.AXE_ERANGE
    ls, ld = B.Layout(s), B.Layout(d)
    assert hc.axe_relayout(C.byref(ls.c), C.byref(ld.c), 2, (C.c_int64 * 2)(128, 256), 2, 0, None, src.size, base.ctypes.data, base.size, None) == B.AXE_EINVAL
    assert hc.axe_relayout(C.byref(ls.c), C.byref(ld.c), 2, (C.c_int64 * 2)(128, 256), 2, 0, src.ctypes.data + 1, src.size, base.ctypes.data, base.size,
                           None) == B.AXE_EINVAL
    right(hc, s, d, (128, 256), src, base)


def test_eval_plans(hc):                                       # noqa: F811
    def ev(spec, n, shape):
        L = B.Layout(spec, ["m"])
        out = np.zeros((max(n, 1), L.E_R, 1), dtype=np.int64)
        rc = hc.axe_layout_eval(C.byref(L.c), len(shape), (C.c_int64 * len(shape))(*shape), n, None, out.ctypes.data, None)
        return rc, out

    for spec, shape in ((W.row_major_spec(6, 10), (6, 10)), (W.row_major_spec(6, 10), (60,)), (W.col_major_spec(6, 10), (6, 10)),
                        (dict(W.col_major_spec(6, 10), O={"m": 5}), (6, 10)), (dict(W.col_major_spec(6, 10), R=[(2, 100, "m")]), (6, 10))):
        for _ in range(2):
            rc, out = ev(spec, 60, shape)
            assert rc == B.AXE_OK and np.array_equal(out, R.evaluate_np(Layout.from_spec(spec), np.arange(60), ["m"]))
        assert ev(spec, 61, shape)[0] == B.AXE_ERANGE and ev(spec, -1, shape)[0] == B.AXE_EINVAL and ev(spec, 0, shape)[0] == B.AXE_OK
        assert ev(spec, 7, (7, 9))[0] == B.AXE_ESHAPE


def test_threads_keep_plans_of_their_own(hc):                  # noqa: F811
    hc.axe_hostcheck_set_buffers(1 << 40, 1 << 40)
    bad = []

    def work(k):
        src = np.arange(64 * 96, dtype=np.uint16)
        s, d = W.row_major_spec(64, 96), W.spec([(64, 1, "m"), (96, 64 + 8 * k, "m")])
        want = np.zeros(96 * (64 + 8 * k), dtype=np.uint16)
        R.relayout_ref(Layout.from_spec(s), Layout.from_spec(d), (64, 96), src, want)
        ls, ld = B.Layout(s), B.Layout(d)
        for _ in range(50):
            dst = np.zeros_like(want)
            rc = hc.axe_relayout(C.byref(ls.c), C.byref(ld.c), 2, (C.c_int64 * 2)(64, 96), 2, 0, src.ctypes.data, src.size, dst.ctypes.data, dst.size, None)
            if rc or not np.array_equal(dst, want):
                bad.append(k)
    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not bad
