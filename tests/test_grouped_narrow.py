"""Grouped GEMM of few rows per group on narrow tiles: which problems take them, what their counted waits rely on, and every input type, epilogue and
tile height against the oracle at the edges of a tile, of a K-tile and of the ring."""
import ctypes as C
import os

import numpy as np
import pytest
import torch

from oracle import axe_ref as R
from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W
from test_gpu_paranoid_build import PARANOID, library
from test_host_plans import hc                                 # noqa: F401


def described(dt, G, M, N, K, gated=False, lda=None, ldb=None, ldc=None, sa=None, sb=None, blocked=False, hint=B.AXE_GROUPED_STREAM):
    lda, ldb, NC = lda or K, ldb or K, N // 2 if gated else N
    ldc = ldc or NC
    n = [(2, 16 * ldb, "m"), (N // 32, 32 * ldb, "m"), (16, ldb, "m")] if gated else [(N, ldb, "m")]
    Bs = W.spec([(G, N * K, "m"), (K // 64, 256 * 64, "m"), (64, 1, "m"), (N // 256, 256 * K, "m"), (256, 64, "m")]) if blocked else \
        W.spec([(G, N * ldb, "m"), (K, 1, "m")] + n)
    code, out = {"bf16": (B.AXE_BF16, B.AXE_BF16), "f16": (B.AXE_F16, B.AXE_F16)}.get(dt, (B.AXE_FP8_E4M3, B.AXE_BF16))
    return B.GroupedGemmDesc(M, N, K, G, B.Layout(W.spec([(M, lda, "m"), (K, 1, "m")])), B.Layout(Bs), B.Layout(W.spec([(M, ldc, "m"), (NC, 1, "m")])),
                             M * lda, G * N * ldb, M * ldc, code, out, epilogue=B.AXE_EPI_SWIGLU if gated else B.AXE_EPI_NONE, kernel_hint=hint,
                             scale_a=sa, scale_b=sb, scale_dtype=B.AXE_SCALE_E8M0 if dt == "fp8 e8m0" else B.AXE_SCALE_F32)


@pytest.mark.parametrize("dt,G,N,K,M,narrow", [                 # (256 compute units assumed where there is no device; M: rows of all groups)
    # 16-bit: more than two tiles per compute unit, and weights that don't stay in the caches or K beyond 512
    ("f16", 128, 1536, 2048, 512, 1), ("f16", 64, 2816, 2048, 64, 1), ("f16", 16, 4096, 4096, 16, 1), ("f16", 128, 1536, 384, 512, 1), ("f16", 128, 1536, 320, 512, 0),
    ("f16", 128, 2048, 768, 16, 0), ("f16", 128, 2048, 768, 17, 1), ("f16", 64, 1536, 512, 512, 0), ("f16", 64, 1536, 576, 512, 1), ("f16", 1, 4096, 4096, 16, 0),
    ("f16", 1024, 256, 1152, 4096, 1), ("f16", 1025, 256, 1152, 4100, 0), ("f16", 4096, 256, 1152, 16384, 0),
    # ... or from nine rows per group on, with short K or few tiles from 13
    ("f16", 8, 1024, 2048, 64, 0), ("f16", 8, 1024, 2048, 65, 1), ("f16", 8, 1024, 768, 96, 0), ("f16", 8, 1024, 768, 97, 1), ("f16", 7, 1024, 1024, 84, 0),
    ("f16", 7, 1024, 1024, 85, 1), ("f16", 4, 512, 1024, 64, 0), ("f16", 4, 512, 1024, 65, 1), ("f16", 64, 1536, 512, 768, 0), ("f16", 64, 1536, 512, 769, 1),
    # fp8: K from 1024, or a tile for a quarter of the compute units, or nine rows per group
    ("fp8", 1, 4096, 4096, 1, 1), ("fp8", 1, 256, 1024, 1, 1), ("fp8", 8, 1024, 2048, 8, 1), ("fp8", 16, 512, 1024, 32, 1), ("fp8", 4, 1024, 768, 4, 1), ("fp8", 4, 768, 768, 4, 0),
    ("fp8", 128, 1024, 896, 3, 0), ("fp8", 128, 1024, 896, 4, 1), ("fp8", 4, 768, 768, 32, 0), ("fp8", 4, 768, 768, 33, 1), ("fp8", 128, 2048, 640, 512, 0),
    ("fp8", 128, 2048, 768, 512, 1), ("fp8", 1024, 256, 1152, 4096, 1), ("fp8", 1025, 256, 1152, 4100, 0)])
def test_which_problems_take_them(hc, dt, G, N, K, M, narrow):   # noqa: F811
    hc.axe_gemm_grouped.argtypes = [C.POINTER(B.axe_gemm_grouped_desc_t)] + [C.c_void_p] * 5
    d = described(dt, G, M, N, K)
    assert hc.axe_gemm_grouped(C.byref(d.c), 1 << 20, 1 << 36, 1 << 44, 1 << 46, None) < 0
    assert hc.axe_hostcheck_grouped_narrow() == narrow
    if dt == "f16" and narrow:                                     # blocked weights stay with the streaming kernel
        d = described(dt, G, M, N, K, blocked=True)
        assert hc.axe_gemm_grouped(C.byref(d.c), 1 << 20, 1 << 36, 1 << 44, 1 << 46, None) < 0
        assert hc.axe_hostcheck_grouped_narrow() == 0


@pytest.mark.parametrize("dt,G,N,K,ldb,rows,height", [            # (rows of all groups together)
    ("fp8", 128, 1536, 2048, 2048, 512, 16), ("fp8", 128, 1536, 2048, 2048, 513, 32), ("fp8", 128, 1536, 2048, 2048, 12 * 128, 32), ("fp8", 128, 1536, 2048, 2048, 12 * 128 + 1, 64),
    ("f16", 128, 1536, 2048, 2048, 1, 32), ("f16", 128, 1536, 2048, 2048, 16 * 128, 32), ("f16", 128, 1536, 2048, 2048, 16 * 128 + 1, 64),
    # rows of B a multiple of 4 KiB apart: from two tiles per compute unit on, with one row per group on average four
    ("fp8", 16, 2048, 4096, 4096, 64, 32), ("fp8", 16, 2048, 4096, 4112, 64, 16), ("fp8", 16, 2048, 2304, 8192, 64, 32), ("fp8", 16, 2048, 6144, 6144, 64, 16),
    ("fp8", 15, 2048, 4096, 4096, 60, 16), ("fp8", 16, 2048, 4096, 4096, 31, 16), ("fp8", 16, 2048, 4096, 4096, 32, 32), ("fp8", 64, 2048, 4096, 4096, 31, 16),
    ("fp8", 64, 2048, 4096, 4096, 32, 32)])
def test_rows_of_a_tile(hc, dt, G, N, K, ldb, rows, height):   # noqa: F811
    hc.axe_gemm_grouped.argtypes = [C.POINTER(B.axe_gemm_grouped_desc_t)] + [C.c_void_p] * 5
    d = described(dt, G, rows, N, K, ldb=ldb)
    assert hc.axe_gemm_grouped(C.byref(d.c), 1 << 20, 1 << 36, 1 << 44, 1 << 46, None) < 0
    assert hc.axe_hostcheck_narrow_rows() == (height if hc.axe_hostcheck_grouped_narrow() else 0)
    assert hc.axe_hostcheck_grouped_narrow() == (0 if dt == "f16" and rows == 1 else 1)


def bodies_of(source, out):
    """The kernels of the narrow tiles, each body by itself: (parameters, whether all its loads of B pass by the caches, lines).  A kernel that goes by its
    table has two bodies, one for either policy, behind each other."""
    import re
    import subprocess
    from paper_2601_19092_amd import build as BLD
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *BLD.FLAGS, "-I", BLD.CSRC, "-S", "--cuda-device-only",
                           os.path.join(BLD.CSRC, source), "-o", str(out)], stderr=subprocess.DEVNULL)
    for m in re.finditer(r"^_ZN3axe5tiles\d+gemm_narrow_(by_table_)?kernelI((?:Li\d+E)+)\w*:[^\n]*\n(.*?)\n\.Lfunc_end", open(out).read(), re.S | re.M):
        lines, pars = m.group(3).split("\n"), [int(x) for x in re.findall(r"Li(\d+)E", m.group(2))]
        tm, tn, wm, wn, nst = pars[2:7]
        ring = nst * (tm + tn) // 8 // (wm * wn)                   # loads of a body before its first counted wait: all stages of the ring
        begins, n = [], 0
        for i, x in enumerate(lines):
            n += bool(re.match(r"\tbuffer_load_dwordx4 .* lds$", x))
            if re.match(r"\ts_waitcnt vmcnt\(\d+\) lgkmcnt\(0\)$", x):
                begins, n = begins + [i] * (n >= ring), 0
        assert len(begins) == (2 if m.group(1) else 1), pars
        ahead = ring + ((tm // wm // 16 + (2 if pars[7] == 2 else 1)) if pars[1] else 0)      # and its first scales
        cuts = [0] + [[i for i, x in enumerate(lines[:b]) if x.startswith("\tbuffer_load_")][-ahead] for b in begins[1:]] + [len(lines)]
        for a, b in zip(cuts, cuts[1:]):
            loads = [x for x in lines[a:b] if re.match(r"\tbuffer_load_dwordx4 .* lds$", x.replace(" nt lds", " lds"))]
            past = sum(" nt lds" in x for x in loads)
            assert past in (0, len(loads) * tn // (tm + tn)), (pars, past)
            yield bool(m.group(1)), pars, past > 0, [x.replace(" nt lds", " lds") for x in lines[a:b]]


def test_loads_between_counted_waits(tmp_path):
    """As for the tile family: no spills, a stage's loads between its counted wait and the next, a trip's scale loads before its first loads; and
    where the table decides, a body for either answer."""
    import re
    seen = []
    for by_table, (dt, sc, tm, tn, wm, wn, nst, grp), past, lines in bodies_of("kernels_gemm_grouped_narrow.hip", tmp_path / "k.s"):
        where = (dt, sc, tm, grp, by_table, past)
        assert not [x for x in lines if "scratch_" in x], where
        # (a descriptor held in vector registers would be read lane by lane, in a loop around every load)
        assert not [i for i, x in enumerate(lines) if "s_cbranch_execnz" in x and any(" lds" in y for y in lines[max(0, i - 12):i])], where
        loads, scales = (tm + tn) // 8 // (wm * wn), (tm // wm // 16 + (2 if grp == 2 else 1)) if sc else 0
        base, u = (nst - 2) * loads, 4 if sc else 2
        first = next(i for i, x in enumerate(lines) if "v_mfma" in x)
        start = next(i for i, x in enumerate(lines) if x.endswith(" lds"))
        last = max(i for i, x in enumerate(lines) if "v_mfma" in x)
        counted = [int(m.group(1)) for x in lines[start:last] for m in [re.match(r"\ts_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)$", x)] if m]
        assert counted[0] == base + loads and sorted(counted[1:]) == sorted(base + (scales if 1 <= k <= nst - 2 else 0) for k in range(u)), (where, counted)
        # between the stages' matrix products the compiler waits for a trip's scales alone, with all loads but the half trip's behind them
        others = [int(m.group(1)) for x in lines[first:last] for m in [re.search(r"vmcnt\((\d+)\)", x)] if m and "lgkmcnt(0)" not in x]
        assert all(n >= 2 * loads for n in others) and (sc or not others), (where, others)
        assert len([x for x in lines if re.match(r"\tbuffer_load_dwordx4 .* lds$", x)]) == (u + nst) * loads, where
        assert len([x for x in lines if re.match(r"\tbuffer_load_(dword|ubyte) ", x)]) == 2 * scales, where
        seen.append(where)
    plain = [w for w in seen if not w[4]]
    assert len(plain) == 30 and not any(w[5] for w in plain)
    assert len({w for w in seen if w[4]}) == 60


# sizes of the groups, N, K-tiles, pitches, rows of a tile
FP8 = [([1, 0, 2, 16, 17, 0, 1, 3] * 2, 2304, 6, 0, 32), ([1, 0, 2, 5, 17, 0, 1, 3] * 2, 2304, 6, 0, 16),   # as many K-tiles as stages
       ([0, 15, 16, 1, 33, 2, 0, 9] * 2, 2304, 7, 1, 32),                   # an odd number of K-tiles, pitches
       ([31, 0, 32, 33, 5, 1, 64, 2], 1024, 16, 0, 64),                     # more rows than the average says
       ([63, 64, 65, 0, 17, 1], 512, 10, 2, 64), ([3, 0] * 70 + [40, 1], 256, 8, 0, 16)]                    # more than 64 groups
F16 = [([16, 0, 33, 1, 32, 17, 2, 15], 2304, 6, 0, 32), ([0, 15, 31, 1, 33, 20, 0, 16], 2304, 7, 1, 32), ([31, 0, 32, 33, 5, 1, 64, 2], 1024, 16, 0, 64),
       ([63, 64, 65, 0, 17, 1], 512, 10, 2, 64), ([30, 0] * 66 + [40, 1], 256, 8, 0, 32)]
SHAPES = [(dt, *s) for dt in ("bf16", "f16") for s in F16] + [(dt, *s) for dt in ("fp8", "fp8 f32", "fp8 e8m0") for s in FP8]


@pytest.mark.parametrize("dt,sizes,N,kt,pads,height", SHAPES)
def test_the_problems_below_take_them(hc, dt, sizes, N, kt, pads, height):   # noqa: F811
    hc.axe_gemm_grouped.argtypes = [C.POINTER(B.axe_gemm_grouped_desc_t)] + [C.c_void_p] * 5
    K, vec = kt * (128 if dt.startswith("fp8") else 64), 16 if dt.startswith("fp8") else 8
    for gated in (False, True):
        d = described(dt, len(sizes), sum(sizes) + 5, N, K, gated, K + vec * pads, K + 2 * vec * pads, (N // 2 if gated else N) + 8 * pads)
        assert hc.axe_gemm_grouped(C.byref(d.c), 1 << 20, 1 << 36, 1 << 44, 1 << 46, None) < 0
        assert (hc.axe_hostcheck_grouped_narrow(), hc.axe_hostcheck_narrow_rows()) == (1, height)


@pytest.mark.gpu
@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("dt,sizes,N,kt,pads,height", SHAPES)
def test_every_row_of_every_group(sizes, N, kt, pads, height, dt, gated):
    fp8 = dt.startswith("fp8")
    K = kt * (128 if fp8 else 64)
    off = np.concatenate([[3], 3 + np.cumsum(sizes)]).astype(np.int32)     # rows 0 .. 2 and the last two belong to no group
    M = int(off[-1]) + 2
    g = W.gemm_grouped_fp8(off, N, K, 70 + K, M=M, scale_dtype="e8m0" if dt == "fp8 e8m0" else "f32") if fp8 else W.gemm_grouped_bf16(off, N, K, 70 + K, M=M, dtype=dt)
    sa = sb = so = None
    if dt in ("fp8 f32", "fp8 e8m0"):
        g.scale_b = g.scale_b / np.float32(K ** 0.5) if dt == "fp8 f32" else (g.scale_b - 5).astype(np.uint8)   # gates around one
        so = [R.e8m0_decode(s).astype(np.float32) if dt == "fp8 e8m0" else s for s in (g.scale_a, g.scale_b)]
        sa, sb = (torch.from_numpy(np.concatenate([s.reshape(-1), np.zeros(-s.size % 4, s.dtype)])).cuda() for s in (g.scale_a, g.scale_b))
    vec = 16 if fp8 else 8
    lda, ldb, NC = K + vec * pads, K + 2 * vec * pads, N // 2 if gated else N
    ldc = NC + 8 * pads

    def image(words, pitch):
        out = np.full((words.shape[0], pitch), 0x7F if fp8 else 0x7FC0, dtype=words.dtype)
        out[:, :K] = words
        return torch.from_numpy(out.view(np.uint8 if fp8 else np.int16)).cuda()

    img = g.b_gnk.reshape(g.G, 2, N // 32, 16, K).transpose(0, 2, 1, 3, 4).reshape(g.G, N, K) if gated else g.b_gnk
    dA, dB, dR = image(g.a_mk, lda), image(img.reshape(g.G * N, K), ldb), torch.from_numpy(g.group_rows).cuda()
    dC = torch.full((M * ldc,), -7, dtype=torch.int16, device="cuda")
    B.axe_gemm_grouped(described(dt, g.G, M, N, K, gated, lda, ldb, ldc, sa, sb), dA, dB, dC, dR)
    torch.cuda.synchronize()
    raw = dC.cpu().numpy().reshape(M, ldc)
    assert (raw[:, NC:] == -7).all() and (raw[:3] == -7).all() and (raw[-2:] == -7).all(), "written outside the groups"
    with library(PARANOID):                                        # the same arithmetic in the same order with a full wait after every load
        dC.fill_(-7)
        B.axe_gemm_grouped(described(dt, g.G, M, N, K, gated, lda, ldb, ldc, sa, sb), dA, dB, dC, dR)
        torch.cuda.synchronize()
    assert np.array_equal(raw, dC.cpu().numpy().reshape(M, ldc))
    code = R.AXE_FP8_E4M3 if fp8 else (R.AXE_BF16 if dt == "bf16" else R.AXE_F16)
    ref = R.gemm_grouped_ref(g.a_mk, g.b_gnk.transpose(0, 2, 1), off, code, **({"scale_a": so[0], "scale_b": so[1]} if so else {}))
    want = R.swiglu_ref(ref) if gated and (not fp8 or so) else (None if gated else ref)
    words = np.ascontiguousarray(raw[:, :NC]).view(np.uint16)
    c = words.view(np.float16).astype(np.float64) if dt == "f16" else R.bf16_to_f64(words)
    if want is None:                                               # unscaled fp8: gates are tens wide, compare where the reference is finite and not tiny
        want = R.swiglu_ref(ref)
    # 16-bit results: 2^-9 / sqrt(3) (bf16) or 2^-12 / sqrt(3) of rounding, fp8 products' own 1.5e-5 besides; a block is a row's 64 values and more
    for e in range(g.G):
        for r0 in range(off[e], off[e + 1], 16):
            rows = slice(r0, min(r0 + 16, off[e + 1]))
            for j in range(0, NC, 64):
                assert R.rel_frobenius(c[rows, j:j + 64], want[rows, j:j + 64]) <= (2e-3 if dt == "f16" else 5e-3), (e, r0, j)
