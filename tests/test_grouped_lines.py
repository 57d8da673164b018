"""fp8 groups with fp32 scales: the last row count per group on average that streams, on both sides of each term of the line."""
import pytest

from test_grouped_choice import S, T, kernel


@pytest.mark.parametrize("G,N,K,last", [
    (128, 1536, 2048, 11), (64, 2816, 2048, 8), (16, 4096, 4096, 8), (64, 1024, 2048, 13),   # the narrow tiles stream, K is long
    (128, 512, 1152, 30), (64, 1024, 768, 24),                                                  # shorter
    (1024, 256, 2048, 36), (1025, 256, 2048, 34), (2048, 256, 2048, 40), (4096, 256, 1152, 76),  # up to 1024 groups they do
    (128, 2048, 512, 19), (64, 1024, 640, 28), (8, 4096, 512, 21), (9, 4096, 512, 17),          # a short pipeline: more than a tile per compute unit, or not
    (16, 256, 8192, 23)])                                                                       # fewer tiles than compute units
def test_last_rows_that_stream(G, N, K, last):
    assert (kernel(G, N, K, last), kernel(G, N, K, last + 1)) == (S, T)
