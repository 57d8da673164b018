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


@pytest.mark.parametrize("G,N,K,stream,tiles", [                # rows per group that still stream, and that take tiles
    (128, 1536, 2048, 8, 12), (128, 2048, 768, 16, 24), (128, 4096, 4096, 5, 9),       # an MoE layer's two products, a larger one
    (128, 512, 1152, 24, 48), (512, 512, 2048, 16, 24), (1024, 512, 1152, 24, 64),     # little weight per group
    (8, 4096, 512, 20, 48), (128, 2048, 512, 16, 32),                                  # a short pipeline
    (8, 1536, 2048, 16, 32), (16, 256, 8192, 9, 24), (32, 512, 640, 48, 96),           # fewer tiles than compute units
    (4096, 256, 1152, 64, 128), (4096, 512, 1024, 48, 96), (2048, 256, 2048, 40, 64)])  # many groups
def test_choice_by_rows_per_group(G, N, K, stream, tiles):
    assert kernel(G, N, K, stream) == S and kernel(G, N, K, tiles) == T
    assert kernel(G, N, K, tiles, B.AXE_GROUPED_STREAM) == S


def test_other_scales_keep_their_lines():
    for rows, want in ((8, S), (9, T)):
        assert kernel(128, 512, 1152, rows, dtype=B.AXE_SCALE_E8M0) == want
