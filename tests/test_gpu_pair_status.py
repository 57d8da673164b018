"""A pair that runs as two launches clears the status word of its workspace, whichever kernels it takes, and leaves the words
around it alone; its results are those of two grouped GEMMs."""
import numpy as np
import pytest
import torch

from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,I", [([1, 0, 0, 2], 256), ([0, 0, 1, 0], 256), ([5, 9, 0, 30], 256), ([400, 0, 3, 90], 384), ([0, 0, 0, 0], 256)])
def test_status_word(sizes, I):
    G, H = len(sizes), 512
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    M = max(int(off[-1]), 3)
    rng = torch.Generator(device="cuda").manual_seed(7)
    x, w1, w2 = (torch.randn(s, generator=rng, device="cuda", dtype=torch.float32).mul_(0.1).to(torch.float16) for s in
                 ((M, H), (G, 2 * I, H), (G, H, I)))
    rows = torch.from_numpy(off).cuda()
    h, c, h2, c2 = (torch.zeros(s, dtype=torch.float16, device="cuda") for s in ((M, I), (M, H)) * 2)
    d1 = B.GroupedGemmDesc(M, 2 * I, H, G, B.Layout(W.row_major_spec(M, H)), B.Layout(W.gated_b_spec(H, 2 * I, G)), B.Layout(W.row_major_spec(M, I)),
                           M * H, w1.numel(), M * I, B.AXE_F16, B.AXE_F16, epilogue=B.AXE_EPI_SWIGLU)
    d2 = B.GroupedGemmDesc(M, H, I, G, B.Layout(W.row_major_spec(M, I)), B.Layout(W.spec([(G, H * I, "m"), (I, 1, "m"), (H, I, "m")])),
                           B.Layout(W.row_major_spec(M, H)), M * I, w2.numel(), M * H, B.AXE_F16, B.AXE_F16)
    room = torch.full((M + 3,), 9, dtype=torch.int32, device="cuda")
    sync = room[1:M + 2]
    for _ in range(3):
        sync[M] = 9
        B.axe_gemm_grouped_pair(d1, d2, x, w1, h, w2, c, rows, sync)
        B.axe_gemm_grouped_pair_status(sync, M)                # raises if the word is not zero
        assert int(room[0]) == 9 and int(room[-1]) == 9
    B.axe_gemm_grouped(d1, x, w1, h2, rows)
    B.axe_gemm_grouped(d2, h2, w2, c2, rows)
    assert torch.equal(h, h2) and torch.equal(c, c2)
