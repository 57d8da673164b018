"""AXE_TILE_MEMBER, the knob that asks for a member of the tile family, is heeded by the very next axe_gemm, whatever plan the thread has
kept, and by every problem that no large tile takes."""
import ctypes as C

import pytest

from paper_2601_19092_amd import binding as B
from test_host_plans import hc                                 # noqa: F401
from test_tile_family import MEMBERS, descriptor, forced


def launched(hc, d):                                           # noqa: F811
    """The member axe_gemm hands to the (absent) device: the stand-ins note it and refuse."""
    hc.axe_gemm.argtypes = [C.POINTER(B.axe_gemm_desc_t), C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p]
    assert hc.axe_gemm(C.byref(d.c), 1 << 20, 1 << 30, 1 << 40, None) < 0
    return hc.axe_hostcheck_gemm_member()


@pytest.mark.parametrize("dt", ["bf16", "fp8"])
def test_one_descriptor_under_changing_members(hc, dt):        # noqa: F811
    d = descriptor(1000, 999, 1024, dt)                       # (edges no large tile serves)
    own = launched(hc, d)
    assert own == 5                                            # 64 x 64
    for m in (7, 0, 8, 0):
        with forced(m):
            assert launched(hc, d) == m
    assert launched(hc, d) == own


@pytest.mark.parametrize("M,N,K,dt", [(256, 256, 256, "bf16"), (64, 64, 64, "bf16"), (512, 512, 128, "f16"), (600, 1500, 320, "bf16"), (512, 512, 128, "fp8")])
def test_short_k_does_not_override_the_knob(hc, M, N, K, dt):  # noqa: F811
    d = descriptor(M, N, K, dt, "f16" if dt == "f16" else "bf16")
    for m, shape in enumerate(MEMBERS):
        with forced(m):
            assert launched(hc, d) == m and B.axe_gemm_describe(d, B.AXE_DESC_C_STORE)[1] == shape[:2]
