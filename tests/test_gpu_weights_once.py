"""Grouped tile kernels whose weights are too many for the last-level cache load them past the caches (where most groups have one row block):
the same bits as half of the groups give, whose weights are few enough for the ordinary loads."""
import pytest
import torch

from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W

G, N, K = 32, 2048, 2304                                           # fp8 151 MB, half of them 75 MB; 16-bit 302 and (a quarter) 75 MB


def describe(M, groups, dt, gated, sa, sb):
    n = [(2, 16 * K, "m"), (N // 32, 32 * K, "m"), (16, K, "m")] if gated else [(N, K, "m")]
    NC = N // 2 if gated else N
    code, out = (B.AXE_FP8_E4M3, B.AXE_BF16) if dt.startswith("fp8") else (B.AXE_BF16, B.AXE_BF16)
    return B.GroupedGemmDesc(M, N, K, groups, B.Layout(W.row_major_spec(M, K)), B.Layout(W.spec([(groups, N * K, "m"), (K, 1, "m")] + n)),
                             B.Layout(W.row_major_spec(M, NC)), M * K, groups * N * K, M * NC, code, out,
                             epilogue=B.AXE_EPI_SWIGLU if gated else B.AXE_EPI_NONE, kernel_hint=0 if dt == "fp8 f32" else B.AXE_GROUPED_TILES_128,
                             scale_a=sa, scale_b=sb, scale_dtype=B.AXE_SCALE_E8M0 if dt == "fp8 e8m0" else B.AXE_SCALE_F32)


@pytest.mark.gpu
@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("dt", ["bf16", "fp8", "fp8 f32", "fp8 e8m0"])
def test_same_bits_as_through_the_caches(dt, gated):
    g = torch.Generator(device="cuda").manual_seed(7)
    sizes = [(40, 128, 1, 0, 129, 17, 64, 90)[i % 8] for i in range(G)]
    rows = torch.tensor([0] + sizes).cumsum(0).to(torch.int32).cuda()
    M = int(rows[-1])
    cast = torch.float8_e4m3fn if dt.startswith("fp8") else torch.bfloat16
    a = torch.empty(M, K, device="cuda").normal_(generator=g).to(cast)
    b = torch.empty(G, N, K, device="cuda").normal_(0, K ** -0.5 * (16 if dt.startswith("fp8") else 1), generator=g).to(cast)
    sa = sb = None
    if dt == "fp8 f32":
        sa, sb = (torch.rand(s, generator=g, device="cuda") + 0.5 for s in ((M, K // 128), (G, N // 128, K // 128)))
    if dt == "fp8 e8m0":
        sa, sb = (torch.randint(124, 130, s, generator=g, device="cuda", dtype=torch.uint8) for s in ((M, K // 128), (G, N // 128, K // 128)))
    NC = N // 2 if gated else N
    step = G // 2 if dt.startswith("fp8") else G // 4
    out = torch.zeros(M, NC, dtype=torch.bfloat16, device="cuda")
    assert B.axe_gemm_grouped_kernel(describe(M, G, dt, gated, sa, sb)) == B.AXE_GROUPED_TILES_128
    B.axe_gemm_grouped(describe(M, G, dt, gated, sa, sb), a, b, out, rows)
    for e in range(0, G, step):
        i, j = int(rows[e]), int(rows[e + step])
        part = torch.zeros(j - i, NC, dtype=torch.bfloat16, device="cuda")
        d = describe(j - i, step, dt, gated, None if sa is None else sa[i:j].contiguous(), None if sb is None else sb[e:e + step].contiguous())
        assert B.axe_gemm_grouped_kernel(d) == B.AXE_GROUPED_TILES_128
        B.axe_gemm_grouped(d, a[i:j].contiguous(), b[e:e + step].contiguous(), part, rows[e:e + step + 1] - rows[e])
        assert torch.equal(out[i:j].view(torch.int16), part.view(torch.int16)), e
        if not gated and sa is None:                               # and they are the product: bf16 results, K terms in fp32
            k = e + 1
            r = slice(int(rows[k]), int(rows[k + 1]))
            want = a[r].float() @ b[k].float().t()
            assert ((out[r].float() - want).norm() / want.norm()).item() <= 5e-3
