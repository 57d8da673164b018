"""fp8 groups with fp32 scales: the last row count per group on average that streams, on both sides of each term of the line."""
import pytest

from test_grouped_choice import S, T, kernel


@pytest.mark.parametrize("G,N,K,last", [
    (128, 1536, 2048, 16), (96, 1024, 1024, 16), (95, 1024, 1024, 16), (64, 1024, 2048, 24), (40, 1024, 1536, 38), (8, 1536, 2048, 128),   # narrow tiles, by tiles per compute unit
    (16, 512, 2048, 192), (16, 256, 8192, 192),                                                        # ... up to 192 rows
    (1024, 256, 2048, 16), (1025, 256, 2048, 6),                                                       # up to 1024 groups
    (128, 1536, 768, 16), (128, 1536, 640, 4),                                                         # from six K-tiles on
    (128, 2048, 512, 4), (512, 256, 512, 15), (2048, 256, 640, 12), (4096, 256, 1152, 8),             # the streaming kernel, by a group's weights
    (8, 4096, 512, 8), (9, 4096, 512, 20), (15, 4096, 512, 8), (16, 4096, 512, 3), (8, 2048, 512, 16), (1, 8192, 640, 21),   # ... and fewer than two tiles per compute unit
    (4096, 512, 1024, 25), (4095, 512, 1024, 6), (4096, 768, 1024, 14), (1024, 2048, 1024, 35)])      # 64 tiles per compute unit and more
def test_last_rows_that_stream(G, N, K, last):
    assert (kernel(G, N, K, last), kernel(G, N, K, last + 1)) == (S, T)
