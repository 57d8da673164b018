"""The grouped GEMM's streaming kernel on problems that are its own: fewer K-tiles than the narrow tiles' ring has stages, blocked weights, more than 1024
groups.  Every variant against the oracle, and the bits of many launches: the split of K over waves adds its partial sums in a fixed order."""
import numpy as np
import pytest
import torch

from oracle import axe_ref as R
from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W
from packing import pack_blocked, pack_gate_up
from routes import narrow_rows

DOZENS = [1, 0, 16, 17, 33, 9, 40, 0, 3, 20, 2, 12]               # K split, 32 rows a pass
# sizes of the groups by the variant that they ask for
SIZES = {"16 rows a pass": [0, 3, 1, 0, 17, 0, 2, 0, 5, 1] * 2, "32 rows a pass": DOZENS, "64 rows a pass, few workgroups": [70, 0, 33, 64, 17],
         "64 rows a pass": [0, 40, 25, 33] * 64}


def problem(dt, sizes, gated, blocked, N=512, tiles=None):
    """Descriptor, device buffers, and the oracle's result."""
    fp8 = dt.startswith("fp8")
    K = (tiles or (8 if blocked else 5)) * (128 if fp8 else 64)
    off = np.concatenate([[0], np.cumsum(sizes)])
    M = int(off[-1]) + 2                                           # the last two rows belong to no group
    scale = {"scale_dtype": "e8m0" if dt == "fp8 e8m0" else "f32"}
    g = W.gemm_grouped_fp8(off, N, K, 31, M=M, **scale) if fp8 else W.gemm_grouped_bf16(off, N, K, 31, M=M, dtype=dt, std_b=2.0 * K ** -0.5)
    sa = sb = so = None
    if " " in dt:
        g.scale_b = g.scale_b / np.float32(K ** 0.5) if dt == "fp8 f32" else (g.scale_b - 5).astype(np.uint8)   # gates around one
        so = [R.e8m0_decode(s).astype(np.float32) if dt == "fp8 e8m0" else s for s in (g.scale_a, g.scale_b)]
        sa, sb = (torch.from_numpy(np.concatenate([s.reshape(-1), np.zeros(-s.size % 4, s.dtype)])).cuda() for s in (g.scale_a, g.scale_b))
    img = pack_gate_up(g.b_gnk) if gated else g.b_gnk
    img = pack_blocked(img) if blocked else img
    Bs = W.gated_b_spec(K, N, g.G, blocked) if gated else (W.blocked_b_spec(K, N, G=g.G) if blocked else W.grouped_gemm_specs(g)[1])
    NC = N // 2 if gated else N
    code = {"bf16": R.AXE_BF16, "f16": R.AXE_F16}.get(dt, R.AXE_FP8_E4M3)
    d = B.GroupedGemmDesc(M, N, K, g.G, B.Layout(W.row_major_spec(M, K)), B.Layout(Bs), B.Layout(W.row_major_spec(M, NC)), M * K, img.size, M * NC,
                          in_dtype=B.AXE_FP8_E4M3 if fp8 else (B.AXE_BF16 if dt == "bf16" else B.AXE_F16), out_dtype=B.AXE_F16 if dt == "f16" else B.AXE_BF16,
                          epilogue=B.AXE_EPI_SWIGLU if gated else B.AXE_EPI_NONE, kernel_hint=B.AXE_GROUPED_STREAM, scale_a=sa, scale_b=sb,
                          scale_dtype=B.AXE_SCALE_E8M0 if dt == "fp8 e8m0" else B.AXE_SCALE_F32)
    ref = R.gemm_grouped_ref(g.a_mk, g.b_gnk.transpose(0, 2, 1), off, code, **({"scale_a": so[0], "scale_b": so[1]} if so else {}))
    words = [torch.from_numpy(np.ascontiguousarray(w.reshape(-1)).view(np.uint8 if fp8 else np.int16)).cuda() for w in (g.a_mk, img)]
    return g, off, d, words, R.swiglu_ref(ref) if gated else ref, NC


@pytest.mark.gpu
@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("variant", list(SIZES))
@pytest.mark.parametrize("dt,blocked", [("bf16", False), ("f16", False), ("bf16", True), ("f16", True), ("fp8", False), ("fp8 f32", False), ("fp8 e8m0", False)])
def test_every_variant(dt, blocked, variant, gated):
    sizes = SIZES[variant]
    if variant == "64 rows a pass" and blocked:
        sizes = sizes[:128]
    g, off, d, (dA, dB), want, NC = problem(dt, sizes, gated, blocked)
    assert narrow_rows(d) == 0
    dC = torch.full((g.M * NC,), -7, dtype=torch.int16, device="cuda")
    B.axe_gemm_grouped(d, dA, dB, dC, torch.from_numpy(g.group_rows).cuda())
    torch.cuda.synchronize()
    raw = dC.cpu().numpy().reshape(g.M, NC)
    assert (raw[-2:] == -7).all(), "written outside the groups"
    words = raw.view(np.uint16)
    c = words.view(np.float16).astype(np.float64) if dt == "f16" else R.bf16_to_f64(words)
    # 16-bit results: 2^-9 / sqrt(3) (bf16) or 2^-12 / sqrt(3) of rounding, fp8 products' own 1.5e-5 besides
    for e in range(g.G):
        for j in range(0, NC, 64):
            rows = slice(off[e], off[e + 1])
            if sizes[e]:
                assert R.rel_frobenius(c[rows, j:j + 64], want[rows, j:j + 64]) <= (2e-3 if dt == "f16" else 5e-3), (e, j)


@pytest.mark.gpu
@pytest.mark.parametrize("dt,blocked,variant", [("bf16", True, "16 rows a pass"), ("f16", True, "32 rows a pass"), ("bf16", True, "64 rows a pass, few workgroups"),
                                                ("fp8 f32", False, "16 rows a pass"), ("fp8 e8m0", False, "32 rows a pass"), ("fp8", False, "64 rows a pass, few workgroups")])
def test_split_sums_are_added_in_a_fixed_order(dt, blocked, variant):
    g, _, d, (dA, dB), _, NC = problem(dt, SIZES[variant], False, blocked, N=1024, tiles=32 if blocked else 5)
    assert narrow_rows(d) == 0
    rows, first = torch.from_numpy(g.group_rows).cuda(), None
    dC = torch.zeros(g.M * NC, dtype=torch.int16, device="cuda")
    for it in range(40):
        dC.zero_()
        B.axe_gemm_grouped(d, dA, dB, dC, rows)
        first = dC.clone() if first is None else first
        assert torch.equal(first, dC), f"launch {it} differs from launch 0 in {(first != dC).sum().item()} elements"


@pytest.mark.gpu
def test_more_than_1024_groups():
    sizes = np.zeros(1100, dtype=np.int64)
    sizes[[0, 63, 64, 700, 1023, 1024, 1099]] = [3, 17, 1, 40, 2, 33, 5]
    g, off, d, (dA, dB), want, NC = problem("bf16", sizes, False, False, N=256, tiles=8)
    assert narrow_rows(d) == 0
    dC = torch.full((g.M * NC,), -7, dtype=torch.int16, device="cuda")
    B.axe_gemm_grouped(d, dA, dB, dC, torch.from_numpy(g.group_rows).cuda())
    torch.cuda.synchronize()
    c = R.bf16_to_f64(dC.cpu().numpy().view(np.uint16).reshape(g.M, NC))
    for e in np.nonzero(sizes)[0]:
        assert R.rel_frobenius(c[off[e]:off[e + 1]], want[off[e]:off[e + 1]]) <= 5e-3, e
