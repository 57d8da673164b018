"""The fused pair where the library takes tiles of 192 rows by itself: several tiles a workgroup and product, so that loads, waits for rows and the publishing
of a tile run on from one tile into the next, on plain weights whose rows are 4 KiB apart (groups start K at places of their own).  Bit for bit
against two launches on tiles of 128 rows (which the oracle checks elsewhere; every height adds a sum up in one order) and against the checking build."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W
from test_gpu_paranoid_build import PARANOID, library
from test_pair_rows import pair_rows

pytestmark = pytest.mark.gpu
SENTINEL = 0x7FC1
# groups, hidden, intermediate, out: 456 tile columns and more in all groups, about 1.4 row blocks each, for 256 workgroups
CASES = {"plain, K 2048": (116, 2048, 512, 2048), "plain, K 512": (228, 512, 256, 512)}


def routed(G, M, seed):
    w = np.exp(np.random.default_rng(seed).normal(0.0, 0.5, G))
    n = np.random.default_rng(seed + 1).multinomial(M, w / w.sum())
    n[3], n[4] = n[3] + n[4], 0                                                            # a group without rows
    return np.concatenate([[0], np.cumsum(n)]).astype(np.int32)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", list(CASES))
def test_tiles_of_192_rows_follow_one_another(case, dtype):
    G, hidden, inter, out = CASES[case]
    M = 184 * G
    assert pair_rows(G, hidden, inter, M) == 192
    off = routed(G, M, 41)
    assert sum(-(-int(n) // 192) for n in np.diff(off)) * (2 * inter // 256) > 256 and sum(-(-int(n) // 192) for n in np.diff(off)) * (out // 256) > 256
    dt, tdt = (B.AXE_F16, torch.float16) if dtype == "f16" else (B.AXE_BF16, torch.bfloat16)
    g = torch.Generator(device="cuda").manual_seed(7)
    a = torch.empty(M * hidden, dtype=tdt, device="cuda").normal_(0.0, 1.0, generator=g)
    w1 = torch.empty(G * 2 * inter * hidden, dtype=tdt, device="cuda").normal_(0.0, 2.0 * hidden ** -0.5, generator=g)
    w2 = torch.empty(G * out * inter, dtype=tdt, device="cuda").normal_(0.0, inter ** -0.5, generator=g)
    rows = torch.from_numpy(off).cuda()

    def run(hint, fused=True):
        d1 = B.GroupedGemmDesc(M, 2 * inter, hidden, G, B.Layout(W.row_major_spec(M, hidden)), B.Layout(W.gated_b_spec(hidden, 2 * inter, G)),
                               B.Layout(W.row_major_spec(M, inter)), a.numel(), w1.numel(), M * inter, dt, dt, epilogue=B.AXE_EPI_SWIGLU, kernel_hint=hint)
        d2 = B.GroupedGemmDesc(M, out, inter, G, B.Layout(W.row_major_spec(M, inter)), B.Layout(W.spec([(G, out * inter, "m"), (inter, 1, "m"), (out, inter, "m")])),
                               B.Layout(W.row_major_spec(M, out)), M * inter, w2.numel(), M * out, dt, dt, kernel_hint=hint)
        assert B.axe_gemm_grouped_pair_fused(d1, d2)
        h = torch.full((M * inter,), SENTINEL, dtype=torch.int16, device="cuda")
        c = torch.full((M * out,), SENTINEL, dtype=torch.int16, device="cuda")
        sync = torch.full((M + 1,), 12345, dtype=torch.int32, device="cuda") if fused else None
        B.axe_gemm_grouped_pair(d1, d2, a, w1, h, w2, c, rows, sync)
        if fused:
            B.axe_gemm_grouped_pair_status(sync, M)
        torch.cuda.synchronize()
        return h, c

    h, c = run(B.AXE_GROUPED_AUTO)
    assert (h != SENTINEL).any() and (c != SENTINEL).any()
    h2, c2 = run(B.AXE_GROUPED_TILES_128, fused=False)
    assert torch.equal(h, h2) and torch.equal(c, c2)
    with library(PARANOID):
        h2, c2 = run(B.AXE_GROUPED_AUTO)
    assert torch.equal(h, h2) and torch.equal(c, c2)
