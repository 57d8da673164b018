"""The family of small and medium GEMM tiles: the layouts axe_gemm_describe reports for each member against the index
functions the kernels compute with, which member a problem takes, and each member on the device against the oracle at the
edges of its tile, of a K-tile and of its ring."""
import ctypes as C
import os

import numpy as np
import pytest
import torch

from oracle import axe_ref as R
from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W

# (tile rows, tile columns, waves of a group, wave columns, groups, stages): tile_family.h
MEMBERS = [(16, 16, 1, 1, 8, 4), (16, 32, 1, 1, 8, 3), (32, 16, 1, 1, 8, 3), (32, 32, 1, 1, 4, 4), (64, 32, 2, 1, 4, 3),
           (64, 64, 4, 2, 2, 4), (128, 64, 8, 2, 1, 5), (128, 128, 8, 2, 1, 4), (256, 128, 8, 2, 1, 3)]
CODE = {"bf16": B.AXE_BF16, "f16": B.AXE_F16, "fp8": B.AXE_FP8_E4M3, "f32": B.AXE_F32}
TOL = {"bf16": 5e-3, "f16": 2e-3, "f32": 3e-5}              # results in 16 bits: their rounding; in fp32: see exact_tolerance


class forced:
    """The library takes this member for every problem it would give to the family (its own knob for experiments)."""

    def __init__(self, member):
        self.member = member

    def __enter__(self):
        os.environ["AXE_TILE_MEMBER"] = str(self.member)

    def __exit__(self, *exc):
        del os.environ["AXE_TILE_MEMBER"]


def descriptor(M, N, K, dt="bf16", out="bf16", scales=None, rows=0, lda=None, ldb=None, ldc=None, off=0):
    lda, ldb, ldc = lda or K, ldb or K, ldc or N
    A = W.spec([(M, lda, "m"), (K, 1, "m")], O={"m": off})
    Bs = W.spec([(K, 1, "m"), (N, ldb, "m")], O={"m": off})
    Cs = W.spec([(M, ldc, "m"), (N, 1, "m")], O={"m": off})
    sa, sb = scales if scales else (None, None)
    return B.GemmDesc(M, N, K, CODE[dt], CODE[out], B.Layout(A), B.Layout(Bs), B.Layout(Cs), M * lda + off, N * ldb + off, M * ldc + off, sa, sb,
                      scale_dtype=B.AXE_SCALE_E8M0 if scales and sa.dtype == torch.uint8 else B.AXE_SCALE_F32, scale_a_rows=rows)


@pytest.mark.parametrize("member", range(len(MEMBERS)))
@pytest.mark.parametrize("dt", ["bf16", "fp8"])
def test_described_layouts_are_the_kernels_index_functions(member, dt):
    hc = C.CDLL(os.environ.get("AXE_TEST_HOST_LIB") or os.path.join(os.path.dirname(B.LIB_PATH), "libaxe_hostcheck.so"))
    fn = hc.axe_hostcheck_describe_vs_tile_maps
    fn.restype = C.c_int
    fn.argtypes = [C.POINTER(B.axe_gemm_desc_t)] + [C.c_int32] * 7 + [C.c_int64, C.c_int32]
    tm, tn, ng, wn, _, _ = MEMBERS[member]
    eb = 1 if dt == "fp8" else 2
    d = descriptor(2 * tm, 2 * tn, 1024, dt)
    with forced(member):
        assert B.axe_gemm_describe(d, B.AXE_DESC_C_STORE)[1] == (tm, tn)
        for which in range(8):
            assert fn(C.byref(d.c), which, tm, tn, 128 // eb, eb, ng, wn, tm * 128 // eb, 2 if tm <= 64 else 0) == 0, which


def taken(M, N, K, dt="bf16"):
    d = descriptor(M, N, K, dt)
    assert B.axe_gemm_tile(d) in (B.AXE_TILE_64x64x32, B.AXE_TILE_256x256x64, B.AXE_TILE_256x224x64)
    return B.axe_gemm_describe(d, B.AXE_DESC_C_STORE)[1]


def test_which_tile_a_problem_takes():
    """The least rows loaded per compute unit over all rounds of tiles (256 compute units assumed where there is no device)."""
    assert taken(16, 3584, 8192) == (16, 16) and taken(1, 512, 8192) == (16, 16)
    assert taken(16, 8192, 8192) == (16, 32)                # 512 tiles of 16 x 16 would take two rounds
    assert taken(64, 3584, 8192) == (32, 32)                # 224 tiles of 64 rows each loaded, against 112 of 96
    assert taken(512, 3584, 8192) == (128, 64)
    assert taken(2000, 2000, 2048) == (128, 128) and taken(1024, 3584, 8192, "fp8") == (128, 128)
    assert taken(2048, 4096, 2048) == (256, 128) and taken(4096, 4096, 2048) == (256, 256)
    assert taken(1000, 1000, 1000) == (64, 64)
    assert taken(256, 256, 256) == (64, 64) and taken(256, 256, 512) == (16, 16)      # the burst variant up to four K-tiles
    # 16-bit inputs, five K-tiles: the 64 x 64 kernel below 2^23 elements of C
    assert taken(2040, 4096, 320) == (64, 64) and taken(2056, 4096, 312) == (256, 128) and taken(1051, 7885, 328) == (256, 128)
    assert taken(1051, 7885, 320) == (64, 64) and taken(1051, 7885, 320, "fp8") == (256, 128)


def operands(M, N, K, dt, scale, rows, seed):
    g = W.gemm_fp8(M, N, K, seed, scaled=False) if dt == "fp8" else (W.gemm_f16 if dt == "f16" else W.gemm_bf16)(M, N, K, seed)
    sa = sb = None
    if scale:
        rng = np.random.default_rng(seed)
        shape_a, shape_b = (M if rows == 1 else -(-M // 128), -(-K // 128)), (-(-N // 128), -(-K // 128))
        draw = (lambda s: rng.integers(120, 135, s).astype(np.uint8)) if scale == "e8m0" else (lambda s: rng.uniform(0.5, 2.0, s).astype(np.float32))
        sa, sb = draw(shape_a), draw(shape_b)
    return g, sa, sb


def padded(words, pitch, off, fill):
    """(rows, K) words at `off` with rows `pitch` apart; what lies between holds `fill`."""
    out = np.full(off + words.shape[0] * pitch, fill, dtype=words.dtype)
    out[off:].reshape(words.shape[0], pitch)[:, :words.shape[1]] = words
    return out


def check(member, M, N, K, dt, out, scale=None, rows=0, pad=0):
    g, sa, sb = operands(M, N, K, dt, scale, rows, 1000 * member + M + N + K)
    t = [None if s is None else torch.from_numpy(s).cuda() for s in (sa, sb)]
    vec = 16 if dt == "fp8" else 8
    off = pad * vec
    lda, ldb, ldc = K + pad * vec, K + 2 * pad * vec, N + (8 * pad if pad < 2 else 3)
    nan = 0x7F if dt == "fp8" else (0x7E00 if dt == "f16" else 0x7FC0)   # read by mistake, it shows
    dA, dB = (torch.from_numpy(padded(w, p, off, nan).view(np.uint8 if dt == "fp8" else np.int16)).cuda() for w, p in ((g.a_mk, lda), (g.b_nk, ldb)))
    d = descriptor(M, N, K, dt, out, tuple(t) if scale else None, rows, lda, ldb, ldc, off)
    dC = torch.full((M * ldc + off,), -7, dtype=torch.float32 if out == "f32" else torch.int16, device="cuda")
    with forced(member):
        assert B.axe_gemm_describe(d, B.AXE_DESC_C_STORE)[1] == MEMBERS[member][:2]
        B.axe_gemm(d, dA, dB, dC)
    torch.cuda.synchronize()
    c = dC.cpu().numpy()
    assert (c[:off] == -7).all()
    c = c[off:].reshape(M, ldc)
    assert (c[:, N:] == -7).all(), "columns past N written"
    c = c[:, :N]
    got = c.astype(np.float64) if out == "f32" else (R.f16_to_f64 if out == "f16" else R.bf16_to_f64)(np.ascontiguousarray(c).view(np.uint16))
    kw = dict(scale_a=sa, scale_b=sb, block_m_a=1) if rows == 1 else dict(scale_a=sa, scale_b=sb)
    if scale == "e8m0":
        kw.update(scale_a=np.exp2(sa.astype(np.float32) - 127).astype(np.float32), scale_b=np.exp2(sb.astype(np.float32) - 127).astype(np.float32))
    want = R.gemm_ref(g.a_mk, g.b_nk.T, {"bf16": R.AXE_BF16, "f16": R.AXE_F16, "fp8": R.AXE_FP8_E4M3}[dt], **(kw if scale else {}))
    # fp32 results: 16-bit inputs sum in fp32 (K at most 1100 here: well below 1e-6); fp8's matrix instruction aligns its
    # products to the largest one, 2^-16 of it (the repository's bound for that case is 3e-5)
    tol = TOL[out] if out != "f32" or dt == "fp8" else 1e-6
    assert R.rel_frobenius(got, want) <= tol
    for r0 in range(0, M, 64):                                     # no tile may hide behind the others
        for c0 in range(0, N, 64):
            assert R.rel_frobenius(got[r0:r0 + 64, c0:c0 + 64], want[r0:r0 + 64, c0:c0 + 64]) <= 4 * tol, (r0, c0)


@pytest.mark.gpu
@pytest.mark.parametrize("member", range(len(MEMBERS)))
@pytest.mark.parametrize("dt,out,scale,rows", [("bf16", "bf16", None, 0), ("f16", "f32", None, 0), ("fp8", "bf16", None, 0), ("fp8", "f32", "f32", 1),
                                               ("fp8", "bf16", "f32", 0), ("fp8", "bf16", "e8m0", 1), ("fp8", "f32", "e8m0", 0)])
def test_member_matches_the_oracle(member, dt, out, scale, rows):
    tm, tn, _, _, wk, nst = MEMBERS[member]
    kt = 128 if dt == "fp8" else 64
    vec = 16 if dt == "fp8" else 8
    # one row and column past whole tiles; K: one chunk past a K-tile, whole trips of the ring plus one, a single chunk
    check(member, 2 * tm + 1, tn + 3, kt + vec, dt, out, scale, rows)
    check(member, tm, 2 * tn + 8, (wk * nst + 1) * kt, dt, out, scale, rows, pad=1)
    check(member, tm - 1, tn - 1, wk * (nst - 1) * kt, dt, out, scale, rows, pad=2)
    # a single chunk of K.  fp8 to fp32: of 16 products the largest
    # is about 3 times the sum's deviation, so an error of 2^-16 of it is 2^-14.4 = 5e-5 of an average sum and more of one that
    # cancels; the 3e-5 of TOL is a norm over many sums of many products, hence 64 columns there
    check(member, 1, (64 if dt == "fp8" and out == "f32" else 1) + member, vec, dt, out, scale, rows)


@pytest.mark.gpu
@pytest.mark.parametrize("member", range(len(MEMBERS)))
def test_fast_build_equals_checking_build(member):
    """Counted waits and one barrier per K-step against a build that waits for every load: the same bits."""
    from test_gpu_paranoid_build import PARANOID, library
    for dt, scale in (("bf16", None), ("fp8", "f32")):
        M, N, K = 520, 392, 2048 + (16 if dt == "fp8" else 8)
        g, sa, sb = operands(M, N, K, dt, scale, 1, 5)
        t = tuple(torch.from_numpy(s).cuda() for s in (sa, sb)) if scale else None
        dA, dB = (torch.from_numpy(np.ascontiguousarray(w).view(np.uint8 if dt == "fp8" else np.int16)).cuda() for w in (g.a_mk, g.b_nk))
        d = descriptor(M, N, K, dt, "bf16", t, 1 if scale else 0)
        out = []
        for path in (B.LIB_PATH, PARANOID):
            with library(path), forced(member):
                out.append(torch.zeros(M * N, dtype=torch.int16, device="cuda"))
                B.axe_gemm(d, dA, dB, out[-1])
                torch.cuda.synchronize()
        assert torch.equal(out[0], out[1])


# ---- grouped: fp8 with fp32 scales on the 128 x 128 tile
def grouped(sizes, N, K, gated, pads=0, seed=0):
    off = np.concatenate([[3], 3 + np.cumsum(sizes)]).astype(np.int32)     # rows 0 .. 2 and the last two belong to no group
    g = W.gemm_grouped_fp8(off, N, K, 700 + seed, M=int(off[-1]) + 2)
    g.scale_b = g.scale_b / np.float32(K ** 0.5)                            # gates around one
    img = g.b_gnk.reshape(g.G, 2, N // 32, 16, K).transpose(0, 2, 1, 3, 4).reshape(g.G, N, K) if gated else g.b_gnk
    lda, ldb, NC = K + 16 * pads, K + 32 * pads, N // 2 if gated else N
    ldc = NC + 8 * pads
    n = [(2, 16 * ldb, "m"), (N // 32, 32 * ldb, "m"), (16, ldb, "m")] if gated else [(N, ldb, "m")]
    Bs = W.spec([(g.G, N * ldb, "m"), (K, 1, "m")] + n)
    dA = torch.from_numpy(padded(g.a_mk, lda, 0, 0x7F)).cuda()
    dB = torch.from_numpy(padded(img.reshape(g.G * N, K), ldb, 0, 0x7F)).cuda()
    sa, sb = torch.from_numpy(g.scale_a).cuda(), torch.from_numpy(g.scale_b).cuda()
    d = B.GroupedGemmDesc(g.M, N, K, g.G, B.Layout(W.spec([(g.M, lda, "m"), (K, 1, "m")])), B.Layout(Bs),
                          B.Layout(W.spec([(g.M, ldc, "m"), (NC, 1, "m")])), dA.numel(), dB.numel(), g.M * ldc, B.AXE_FP8_E4M3, B.AXE_BF16,
                          epilogue=B.AXE_EPI_SWIGLU if gated else B.AXE_EPI_NONE, scale_a=sa, scale_b=sb)
    return g, off, d, dA, dB, torch.from_numpy(g.group_rows).cuda(), ldc, NC


def test_grouped_choice_and_layouts():
    class Fake:
        def data_ptr(self):
            return 4096

    def kernel(M, K, N=512, G=4, hint=0):
        d = B.GroupedGemmDesc(M, N, K, G, B.Layout(W.row_major_spec(M, K)), B.Layout(W.spec([(G, N * K, "m"), (K, 1, "m"), (N, K, "m")])),
                              B.Layout(W.row_major_spec(M, N)), M * K, G * N * K, M * N, B.AXE_FP8_E4M3, B.AXE_BF16, kernel_hint=hint,
                              scale_a=Fake(), scale_b=Fake())
        return B.axe_gemm_grouped_kernel(d), d
    S, T = B.AXE_GROUPED_STREAM, B.AXE_GROUPED_TILES_128
    assert kernel(8 * 4, 2048)[0] == S and kernel(8 * 4 + 1, 2048)[0] == T
    assert kernel(17 * 4, 768)[0] == S and kernel(17 * 4 + 1, 768)[0] == T
    assert kernel(4000, 384)[0] == S and kernel(4000, 512)[0] == T           # fewer K-tiles than the ring has stages
    assert kernel(4000, 2048, hint=B.AXE_GROUPED_STREAM)[0] == S
    with pytest.raises(B.AxeError):
        kernel(4000, 2048, hint=B.AXE_GROUPED_TILES)
    d = kernel(4000, 2048)[1]
    dense = descriptor(1024, 4096, 2048, "fp8")
    with forced(7):
        for which in (B.AXE_DESC_A_G2L_THREADS, B.AXE_DESC_B_LDS, B.AXE_DESC_A_OPERAND, B.AXE_DESC_C_STORE):
            assert B.axe_gemm_grouped_describe(d, which) == B.axe_gemm_describe(dense, which)


@pytest.mark.gpu
@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("sizes,N,K,pads", [([0, 1, 127, 128, 129, 0, 300, 16], 256, 512, 0),     # as many K-tiles as stages; edges of a tile
                                            ([257, 0, 40, 64], 512, 640, 1),                      # an odd number of K-tiles, pitches
                                            ([200] * 3 + [0] * 70 + [385, 90] * 4, 768, 768, 0),  # more than 64 groups; a trip of two stages
                                            ([130, 5] * 150, 512, 1152, 0)])                      # several tiles per workgroup, one stage past two trips
def test_grouped_matches_the_oracle(sizes, N, K, pads, gated):
    g, off, d, dA, dB, dR, ldc, NC = grouped(sizes, N, K, gated, pads)
    assert B.axe_gemm_grouped_kernel(d) == B.AXE_GROUPED_TILES_128
    dC = torch.full((g.M * ldc,), -7, dtype=torch.int16, device="cuda")
    B.axe_gemm_grouped(d, dA, dB, dC, dR)
    torch.cuda.synchronize()
    raw = dC.cpu().numpy().reshape(g.M, ldc)
    assert (raw[:, NC:] == -7).all() and (raw[:3] == -7).all() and (raw[-2:] == -7).all(), "written outside the groups"
    ref = R.gemm_grouped_ref(g.a_mk, g.b_gnk.transpose(0, 2, 1), off, R.AXE_FP8_E4M3, scale_a=g.scale_a, scale_b=g.scale_b)
    want = R.swiglu_ref(ref) if gated else ref
    c = R.bf16_to_f64(np.ascontiguousarray(raw[:, :NC]).view(np.uint16))
    # bf16 results: 2^-9 / sqrt(3) = 1.1e-3 of rounding (measured 1.7e-3 with the fp8 products' own); one row is a few hundred values
    for e in range(g.G):
        for r0 in range(off[e], off[e + 1], 16):
            rows = slice(r0, min(r0 + 16, off[e + 1]))
            for j in range(0, NC, 64):
                assert R.rel_frobenius(c[rows, j:j + 64], want[rows, j:j + 64]) <= 5e-3, (e, r0, j)


@pytest.mark.gpu
def test_grouped_fast_build_equals_checking_build_and_every_replay():
    from test_gpu_paranoid_build import PARANOID, library
    g, off, d, dA, dB, dR, ldc, NC = grouped([130, 5] * 150, 512, 1152, True)
    out = []
    for path in (B.LIB_PATH, PARANOID):
        with library(path):
            for _ in range(3):
                out.append(torch.zeros(g.M * ldc, dtype=torch.int16, device="cuda"))
                B.axe_gemm_grouped(d, dA, dB, out[-1], dR)
        torch.cuda.synchronize()
    assert all(torch.equal(out[0], o) for o in out[1:])


# ---- what the counted waits rely on, on the ISA hipcc emits
def kernels_of(source, out):
    import re
    import subprocess
    from paper_2601_19092_amd import build as BLD
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *BLD.FLAGS, "-I", BLD.CSRC, "-S", "--cuda-device-only",
                           os.path.join(BLD.CSRC, source), "-o", str(out)], stderr=subprocess.DEVNULL)
    for m in re.finditer(r"^_ZN3axe5tiles17gemm_tiles_kernelI((?:Li\d+E)+)\w*:[^\n]*\n(.*?)\n\ts_endpgm", open(out).read(), re.S | re.M):
        yield [int(x) for x in re.findall(r"Li(\d+)E", m.group(1))], m.group(2).split("\n")


@pytest.mark.parametrize("source", ["kernels_gemm_tiles_16bit.hip", "kernels_gemm_tiles_fp8.hip", "kernels_gemm_tiles_grouped.hip"])
def test_loads_between_counted_waits(source, tmp_path):
    """In every K loop: no spills, each stage's loads between its counted wait and the next, the scale loads of a trip after its
    first wait and before that stage's loads, and no wait of the compiler's own that is stricter than the counted ones."""
    import re
    seen = 0
    for (dt, sc, tm, tn, wm, wn, wk, nst, grp), lines in kernels_of(source, tmp_path / "k.s"):
        assert not [x for x in lines if "scratch_" in x], (dt, sc, tm, tn, grp)
        loads = tm // 8 // (wm * wn) + tn // 8 // (wm * wn)
        scales = (tm // wm // 16 + (2 if grp == 2 else 1)) if sc else 0
        base = (nst - 2) * loads
        labels = {x.split(":")[0]: i for i, x in enumerate(lines) if re.match(r"^\.LBB\d+_\d+:", x)}
        loops = [(labels[m.group(1)], i) for i, x in enumerate(lines) for m in [re.match(r"\ts_cbranch_\w+ (\.LBB\d+_\d+)", x)]
                 if m and labels.get(m.group(1), i) < i]
        loops = [a for a in loops if any("v_mfma" in x for x in lines[a[0]:a[1]])]
        inner = [a for a in loops if not any(b != a and a[0] <= b[0] and b[1] <= a[1] for b in loops)]
        assert inner
        for a, b in inner:
            tokens = []
            for x in lines[a:b]:
                if m := re.match(r"\ts_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)$", x):
                    tokens.append(int(m.group(1)))
                elif re.match(r"\tbuffer_load_dwordx4 .* lds$", x):
                    tokens.append("L")
                elif re.match(r"\tbuffer_load_(dword|ubyte) ", x):
                    tokens.append("S")
                elif m := re.search(r"vmcnt\((\d+)\)", x):
                    assert int(m.group(1)) >= base, (dt, sc, tm, tn, grp, x)
            waits = [t for t in tokens if isinstance(t, int)]
            text = "".join("W" if isinstance(t, int) else t for t in tokens)
            u = 4 if sc else 2
            assert waits == [base + (scales if 1 <= k <= nst - 2 else 0) for k in range(u)], (dt, sc, tm, tn, grp, waits)
            # (grouped loops are rotated by the branch of a half trip: their text may begin inside a stage)
            if grp == 0:
                assert text == "W" + "S" * scales + "L" * loads + ("W" + "L" * loads) * (u - 1), (dt, sc, tm, tn, text)
            else:
                assert text.count("L") == u * loads and text.count("S") == scales and "LS" not in text, (sc, tm, tn, text)
            seen += 1
    assert seen >= (2 if "grouped" in source else 18)
