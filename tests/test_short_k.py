"""Which kernel a GEMM of a few K-tiles takes, at points where the 64 x 64 kernel and the cheapest member of the tile family were timed."""
import pytest

from test_forced_member import launched
from test_host_plans import hc                                 # noqa: F401
from test_tile_family import descriptor

SMALL = -1                                                     # the 64 x 64 kernel


@pytest.mark.parametrize("dt,M,N,K,small", [
    # fp8: one K-tile and one round of 64 x 64 tiles
    ("fp8", 128, 4096, 128, True), ("fp8", 1, 8192, 64, True), ("fp8", 1000, 1000, 128, True), ("fp8", 1000, 1100, 128, False), ("fp8", 128, 4096, 144, False),
    # 16-bit inputs, the burst variant
    ("bf16", 1024, 768, 384, True), ("bf16", 128, 8192, 448, True), ("bf16", 512, 768, 512, True), ("bf16", 512, 512, 384, True), ("bf16", 512, 512, 512, False),
    ("bf16", 256, 256, 384, False), ("bf16", 256, 256, 320, True), ("f16", 64, 2048, 384, True), ("f16", 64, 2048, 448, False), ("bf16", 1024, 1024, 576, False),
    # up to five K-tiles: large members where they nearly fill one round
    ("bf16", 60000, 90, 192, False), ("bf16", 20000, 380, 256, False), ("bf16", 2500, 2501, 320, False), ("f16", 2500, 2501, 288, False),
    ("f16", 3072, 2048, 288, True), ("bf16", 3072, 2048, 192, True), ("bf16", 1024, 6144, 288, True), ("f16", 768, 4096, 256, True),
    ("bf16", 3840, 1279, 288, True), ("bf16", 1051, 7885, 288, True), ("bf16", 500, 1500, 320, True), ("bf16", 2040, 4090, 320, True)])
def test_small_kernel_or_family(hc, dt, M, N, K, small):       # noqa: F811
    d = descriptor(M, N, K, dt, "f16" if dt == "f16" else "bf16")
    assert (launched(hc, d) == SMALL) == small
