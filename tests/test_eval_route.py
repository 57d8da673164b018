"""Evaluations with replicas: by blocks of indices, or on the general kernel where a few indices have an odd number of words that
wastes half of a block's trips -- and the values either way (host stand-in; the kernels: tests/test_gpu_eval_replicas.py)."""
import ctypes as C

import numpy as np
import pytest

from oracle import axe_ref as R
from oracle.axe_layout import Layout
from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W
from test_host_plans import hc                                 # noqa: F401


@pytest.mark.parametrize("rows,cols,replicas,axes,blocks", [
    (32, 48, 43, 3, 0), (100, 100, 43, 3, 0), (100, 100, 47, 3, 0), (300, 301, 43, 3, 1),      # 129 and 141 words: half trips
    (32, 48, 129, 1, 1), (32, 48, 42, 3, 1), (32, 48, 57, 3, 1), (32, 48, 17, 3, 1), (32, 48, 128, 2, 1), (32, 48, 129, 2, 0)])
def test_by_blocks_or_not(hc, rows, cols, replicas, axes, blocks):   # noqa: F811
    names = ["a", "b", "c"][:axes]
    spec = W.spec([(rows, 3, names[0]), (cols, 1, names[-1])], R=[(replicas, 5000, names[axes // 2])])
    L = B.Layout(spec, names)
    n = rows * cols
    room = np.zeros(n * replicas * axes + 2, dtype=np.int64)
    out = room[(-room.ctypes.data % 16) // 8:][:n * replicas * axes]
    assert hc.axe_layout_eval(C.byref(L.c), 2, (C.c_int64 * 2)(rows, cols), n, None, out.ctypes.data, None) == B.AXE_OK
    assert hc.axe_hostcheck_eval_by_blocks() == blocks
    k = np.arange(0, n, 97)
    assert np.array_equal(out.reshape(n, replicas, axes)[k], R.evaluate_np(Layout.from_spec(spec), k, names))
