"""The tile table of the grouped tile kernels at the group counts where it changes its way: up to 64 groups, up to 128 (both halves fetched
at once), beyond; with empty groups at either end of a half, and more tiles than one round of workgroups."""
import numpy as np
import pytest
import torch

from oracle import axe_ref as R
from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W


def sizes_of(G, seed):
    rng = np.random.default_rng(seed)
    n = rng.integers(0, 300, G) * (rng.random(G) < 0.6)
    n[[i for i in (0, 63, 64, 127, 128, G - 1) if i < G]] = 0
    n[G // 2] = 257
    return n


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", [B.AXE_GROUPED_TILES_128, B.AXE_GROUPED_TILES_256])
@pytest.mark.parametrize("G", [1, 63, 64, 65, 127, 128, 129, 193])
def test_every_tile_of_every_group(G, kernel):
    off = np.concatenate([[2], 2 + np.cumsum(sizes_of(G, G))]).astype(np.int32)
    g = W.gemm_grouped_bf16(off, 512, 256, 40 + G, M=int(off[-1]) + 3)
    As, Bs, Cs = W.grouped_gemm_specs(g)
    dA, dB = (torch.from_numpy(w.view(np.int16).copy()).cuda().reshape(-1) for w in (g.a_mk, g.b_gnk))
    dR = torch.from_numpy(g.group_rows).cuda()
    dC = torch.full((g.M * g.N,), -7, dtype=torch.int16, device="cuda")
    d = B.GroupedGemmDesc(g.M, g.N, g.K, g.G, B.Layout(As), B.Layout(Bs), B.Layout(Cs), g.a_mk.size, g.b_gnk.size, g.M * g.N, kernel_hint=kernel)
    B.axe_gemm_grouped(d, dA, dB, dC, dR)
    torch.cuda.synchronize()
    raw = dC.cpu().numpy().reshape(g.M, g.N)
    assert (raw[:2] == -7).all() and (raw[-3:] == -7).all(), "written outside the groups"
    ref = R.gemm_grouped_ref(g.a_mk, g.b_gnk.transpose(0, 2, 1), off, R.AXE_BF16)
    c = R.bf16_to_f64(np.ascontiguousarray(raw).view(np.uint16))
    for e in range(G):                                             # bf16 results: 2^-9 / sqrt(3) of rounding, 128 and more values
        for j in range(0, g.N, 256):
            rows = slice(off[e], off[e + 1])
            if off[e + 1] > off[e]:
                assert R.rel_frobenius(c[rows, j:j + 256], ref[rows, j:j + 256]) <= 5e-3, (e, j)


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", [B.AXE_GROUPED_TILES_128, B.AXE_GROUPED_TILES_256])
@pytest.mark.parametrize("dt,K,ldb", [("bf16", 64, 2048), ("bf16", 256, 2048), ("f16", 320, 2048), ("bf16", 640, 4096), ("f16", 2048, 2048)])
def test_k_tiles_from_a_place_of_the_groups_own(dt, K, ldb, kernel):
    """Rows of B a multiple of 4 KiB apart: every group starts K at another K-tile and comes round (1, 4, 5, 10 and 32 K-tiles)."""
    off = np.concatenate([[0], np.cumsum([130, 1, 0, 40, 300, 17, 128, 5])]).astype(np.int32)
    g = W.gemm_grouped_bf16(off, 256, K, 90 + K, dtype=dt)
    img = np.full((g.G * g.N, ldb), 0x7FC0 if dt == "bf16" else 0x7E00, dtype=np.uint16)      # what lies between the rows is never multiplied
    img[:, :K] = g.b_gnk.reshape(g.G * g.N, K)
    dA, dB = (torch.from_numpy(w.view(np.int16).copy()).cuda().reshape(-1) for w in (g.a_mk, img))
    dC = torch.full((g.M * g.N,), -7, dtype=torch.int16, device="cuda")
    code = B.AXE_BF16 if dt == "bf16" else B.AXE_F16
    d = B.GroupedGemmDesc(g.M, g.N, K, g.G, B.Layout(W.row_major_spec(g.M, K)), B.Layout(W.spec([(g.G, g.N * ldb, "m"), (K, 1, "m"), (g.N, ldb, "m")])),
                          B.Layout(W.row_major_spec(g.M, g.N)), g.M * K, img.size, g.M * g.N, code, code, kernel_hint=kernel)
    B.axe_gemm_grouped(d, dA, dB, dC, torch.from_numpy(g.group_rows).cuda())
    torch.cuda.synchronize()
    words = dC.cpu().numpy().reshape(g.M, g.N).view(np.uint16)
    c = R.bf16_to_f64(words) if dt == "bf16" else words.view(np.float16).astype(np.float64)
    ref = R.gemm_grouped_ref(g.a_mk, g.b_gnk.transpose(0, 2, 1), off, R.AXE_BF16 if dt == "bf16" else R.AXE_F16)
    for e in range(g.G):
        rows = slice(off[e], off[e + 1])
        if off[e + 1] > off[e]:                                    # 16-bit results: 2^-9 / sqrt(3) of rounding at most
            assert R.rel_frobenius(c[rows], ref[rows]) <= (5e-3 if dt == "bf16" else 2e-3), e
