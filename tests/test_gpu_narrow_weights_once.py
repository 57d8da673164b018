"""Narrow tiles with more weights than stay in the last-level cache: the table decides how B is loaded, past the caches where most groups have one row
block, through them elsewhere.  Either way the bits of slices of the groups, whose weights are few enough for the ordinary loads, and the product."""
import ctypes as C

import pytest
import torch

from paper_2601_19092_amd import binding as B
from test_gpu_paranoid_build import PARANOID, library
from test_grouped_narrow import described
from test_host_plans import hc                                 # noqa: F401

G, N, K = 32, 2048, 2304                                           # fp8 151 MB, half of them 75 MB; 16-bit 302 and (a quarter) 75 MB
SIZES = {"16 rows": [1, 0, 5, 16, 2, 3, 0, 4], "32 rows": [20, 0, 32, 5, 1, 12, 9, 10], "64 rows": [40, 64, 1, 0, 30, 17, 20, 33],   # one row block each
         "16 rows, blocks": [0, 0, 0, 31, 0, 0, 0, 0], "32 rows, blocks": [0, 0, 0, 89, 0, 0, 0, 0], "64 rows, blocks": [0, 2, 0, 0, 0, 203, 0, 0]}
CASES = [(dt, which) for dt in ("bf16", "f16", "fp8", "fp8 f32", "fp8 e8m0") for which in SIZES if dt.startswith("fp8") or not which.startswith("16")]


def case(dt, which):
    sizes = SIZES[which] * (G // 8)
    return sizes, (G // 2 if dt.startswith("fp8") else G // 4), sum(sizes)


class Fake:
    def data_ptr(self):
        return 1 << 20


@pytest.mark.parametrize("dt,which", CASES)
def test_they_take_the_narrow_tiles(hc, dt, which):            # noqa: F811
    hc.axe_gemm_grouped.argtypes = [C.POINTER(B.axe_gemm_grouped_desc_t)] + [C.c_void_p] * 5
    _, part, M = case(dt, which)
    for groups in (G, part) if dt.startswith("fp8") else (G,):
        scale = Fake() if " " in dt else None
        d = described(dt, groups, M * groups // G, N, K, sa=scale, sb=scale)
        assert hc.axe_gemm_grouped(C.byref(d.c), 1 << 20, 1 << 36, 1 << 44, 1 << 46, None) < 0
        assert hc.axe_hostcheck_grouped_narrow() == 1


@pytest.mark.gpu
@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("dt,which", CASES)
def test_bits_of_slices_and_the_product(dt, which, gated):
    fp8 = dt.startswith("fp8")
    sizes, part, M = case(dt, which)
    g = torch.Generator(device="cuda").manual_seed(7)
    rows = torch.tensor([0] + sizes).cumsum(0).to(torch.int32).cuda()
    cast = torch.float8_e4m3fn if fp8 else (torch.bfloat16 if dt == "bf16" else torch.float16)
    a = torch.empty(M, K, device="cuda").normal_(generator=g).to(cast)
    b = torch.empty(G, N, K, device="cuda").normal_(0, K ** -0.5 * (16 if fp8 else 1), generator=g).to(cast)
    sa = sb = fa = fb = None
    if dt == "fp8 f32":
        sa, sb = (torch.rand(s, generator=g, device="cuda") + 0.5 for s in ((M, K // 128), (G, N // 128, K // 128)))
        fa, fb = sa.double(), sb.double()
    if dt == "fp8 e8m0":
        sa, sb = (torch.randint(124, 130, s, generator=g, device="cuda", dtype=torch.uint8) for s in ((M, K // 128), (G, N // 128, K // 128)))
        fa, fb = (torch.exp2(s.double() - 127) for s in (sa, sb))
    NC = N // 2 if gated else N

    def whole_words(s):                                            # E8M0 codes are read in whole 4-byte words
        return None if s is None else torch.cat([s.reshape(-1), s.new_zeros(4)])

    def run(i, j, e, groups):
        out = torch.zeros(j - i, NC, dtype=torch.float16 if dt == "f16" else torch.bfloat16, device="cuda")
        scales = (None, None) if sa is None else (whole_words(sa[i:j]), whole_words(sb[e:e + groups]))
        d = described(dt, groups, j - i, N, K, gated, sa=scales[0], sb=scales[1])
        B.axe_gemm_grouped(d, a[i:j].contiguous(), b[e:e + groups].contiguous(), out, rows[e:e + groups + 1] - rows[e])
        torch.cuda.synchronize()
        return out

    out = run(0, M, 0, G)
    with library(PARANOID):                                        # the same arithmetic in the same order with a full wait after every load
        assert torch.equal(out.view(torch.int16), run(0, M, 0, G).view(torch.int16))
    if fp8:                                                        # (16-bit slices of few rows may go to the streaming kernel, whose sums have another order)
        for e in range(0, G, part):
            i, j = int(rows[e]), int(rows[e + part])
            assert torch.equal(out[i:j].view(torch.int16), run(i, j, e, part).view(torch.int16)), e
    for e in range(G):
        i, j = int(rows[e]), int(rows[e + 1])
        if i == j:
            continue
        x, w = a[i:j].double(), b[e].double()
        if fa is not None:
            x = x * fa[i:j].repeat_interleave(128, 1)
            scale = fb[e].repeat_interleave(128, 1)                # a row per 128 columns of the logical B, whose gate and up halves lie in runs of 16
            if gated:
                w = w.reshape(N // 32, 2, 16, K).transpose(0, 1).reshape(N, K)
            w = w * scale.repeat_interleave(128, 0)
        elif gated:
            w = w.reshape(N // 32, 2, 16, K).transpose(0, 1).reshape(N, K)
        p = x @ w.t()
        want = torch.nn.functional.silu(p[:, :NC]) * p[:, NC:] if gated else p
        err = ((out[i:j].double() - want).norm() / want.norm()).item()
        # results of 16 bits (2^-9 / sqrt(3) in bf16, 2^-12 / sqrt(3) in fp16), thousands of values; fp8 products' own 1.5e-5 besides
        assert err <= (1e-3 if dt == "f16" else 3e-3), (e, err)
