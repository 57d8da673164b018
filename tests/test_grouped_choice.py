"""fp8 groups with fp32 scales: which kernel AUTO takes, at points where both were timed.  Hints are heeded whatever the sizes."""
import pytest

from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W

S, T = B.AXE_GROUPED_STREAM, B.AXE_GROUPED_TILES_128


class Fake:
    def data_ptr(self):
        return 4096


def kernel(G, N, K, rows, hint=B.AXE_GROUPED_AUTO, dtype=B.AXE_SCALE_F32):
    M = G * rows
    d = B.GroupedGemmDesc(M, N, K, G, B.Layout(W.row_major_spec(M, K)), B.Layout(W.spec([(G, N * K, "m"), (K, 1, "m"), (N, K, "m")])),
                          B.Layout(W.row_major_spec(M, N)), M * K, G * N * K, M * N, B.AXE_FP8_E4M3, B.AXE_BF16, kernel_hint=hint,
                          scale_a=Fake(), scale_b=Fake(), scale_dtype=dtype)
    return B.axe_gemm_grouped_kernel(d)


# Rows per group that still stream, and that take tiles; both timed, with weights out of the caches: streaming over tiles at either (us where they tell more)
@pytest.mark.parametrize("G,N,K,stream,tiles", [
    (128, 1536, 2048, 16, 20),        # 0.98, 1.04: an MoE layer's two products, a larger one
    (128, 2048, 768, 16, 24),         # 0.98, 1.05
    (128, 4096, 4096, 16, 20),        # 1.01, 1.05
    (64, 2816, 2048, 16, 24),         # 0.98, 1.06
    (128, 512, 1152, 24, 112),        # 1.05 (level from 16 to 96 rows), 1.14: little weight per group
    (512, 512, 2048, 16, 24),         # 1.01, 1.06
    (1024, 512, 1152, 16, 24),        # 1.02, 1.04
    (1024, 256, 1024, 16, 40),        # 1.02, 1.07; at 64 rows 103 / 80 us
    (8, 4096, 512, 8, 12),            # 0.99, 1.03: a short pipeline (the streaming kernel itself)
    (128, 2048, 512, 4, 8),           # 1.04, 1.11; at 24 rows 49 / 32 us
    (512, 256, 512, 14, 18),          # 0.96, 1.05
    (9, 4096, 512, 20, 24),           # 0.98, 1.07: fewer than two tiles per compute unit
    (32, 512, 640, 10, 20),           # 1.00, 1.29
    (8, 1536, 2048, 96, 160),         # 0.96, 1.15: fewer tiles than compute units
    (32, 512, 2048, 96, 112),         # 0.98, 1.13
    (4096, 256, 1152, 8, 16),         # 0.92, 1.08: many groups; at 64 rows 684 / 400 us
    (2048, 256, 2048, 6, 9),          # 1.01, 1.15; at 40 rows twice
    (4096, 512, 1024, 24, 28),        # 0.92, 1.02: more workgroups of tiles than run at once
    (4096, 768, 1024, 12, 20)])       # 1.00, 1.15
def test_choice_by_rows_per_group(G, N, K, stream, tiles):
    assert kernel(G, N, K, stream) == S and kernel(G, N, K, tiles) == T
    assert kernel(G, N, K, tiles, B.AXE_GROUPED_STREAM) == S


def test_other_scales_keep_their_lines():
    for rows, want in ((8, S), (9, T)):
        assert kernel(128, 512, 1152, rows, dtype=B.AXE_SCALE_E8M0) == want
