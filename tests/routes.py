"""Which of the two kernels that stream a grouped GEMM's weights a problem takes (helper; axe_gemm_grouped_kernel answers AXE_GROUPED_STREAM for both)."""
import ctypes as C
import os

from paper_2601_19092_amd import binding as B

_lib = None


def narrow_rows(desc):
    """Rows of the narrow tiles that a problem which streams takes, 0: the streaming kernel.  Asked of the host layer over stand-ins of the kernels: nothing is
    launched, and the addresses are made up."""
    global _lib
    if _lib is None:
        path = os.path.join(os.path.dirname(B.LIB_PATH), "libaxe_hostcheck.so")
        if not os.path.exists(path):
            from paper_2601_19092_amd.build import build_hostcheck
            build_hostcheck()
        _lib = C.CDLL(path)
        _lib.axe_gemm_grouped.argtypes = [C.POINTER(B.axe_gemm_grouped_desc_t)] + [C.c_void_p] * 5
    assert B.axe_gemm_grouped_kernel(desc) == B.AXE_GROUPED_STREAM
    assert _lib.axe_gemm_grouped(C.byref(desc.c), 1 << 20, 1 << 36, 1 << 44, 1 << 46, None) < 0      # (the stand-in answers that it has no device)
    return _lib.axe_hostcheck_narrow_rows()
