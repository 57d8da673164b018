"""Timing cases of the library: what a user's program has it do, over the range of sizes, types and layouts it accepts.

Five kinds of case, each through the entry points of paper_2601_19092_amd.binding:

  gemm      axe_gemm: one linear layer, C = A B, from a decode step (a handful of rows) through prefill chunks to 8192^3;
            bf16 and fp16 with a 16-bit or an fp32 result, fp8 unscaled or with fp32 / E8M0 scales per 128 x 128 block or
            per row and 128-wide k block of A
  moe       the expert computation of a mixture-of-experts layer: in 16 bits one axe_gemm_grouped_pair, in fp8 two
            axe_gemm_grouped calls on quantised activations (quantising between them is the caller's business)
  relayout  axe_relayout between two layouts of one matrix
  eval      axe_layout_eval of a layout at every logical index or at given ones

Inputs come from the seed alone and are made on the GPU.
"""
from __future__ import annotations

import math

import torch

from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W

HIDDEN, INTER, EXPERTS, TOPK = W.MOE_HIDDEN, W.MOE_INTER, W.MOE_EXPERTS, W.MOE_TOPK
TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "fp8": torch.float8_e4m3fn, "f32": torch.float32}
CODE = {"bf16": B.AXE_BF16, "f16": B.AXE_F16, "fp8": B.AXE_FP8_E4M3, "f32": B.AXE_F32}
WORDS = {1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}


def listed():
    return [
        # the smallest dense call: configuration 1, where the launch and the host call count
        {"name": "gemm bf16 256^3 f32 out", "kind": "gemm", "dtype": "bf16", "out": "f32", "scales": "none", "M": 256, "N": 256, "K": 256},
        # a decode step through the tensor-parallel shard of configuration 4: 16 rows against 3584 x 8192 weights
        {"name": "gemm bf16 decode 16 rows", "kind": "gemm", "dtype": "bf16", "out": "bf16", "scales": "none", "M": 16, "N": 3584, "K": 8192},
        # an ordinary fp16 product with edges that fill no tile
        {"name": "gemm f16 2000x2000x2048", "kind": "gemm", "dtype": "f16", "out": "f16", "scales": "none", "M": 2000, "N": 2000, "K": 2048},
        # configuration 3: the largest dense product
        {"name": "gemm bf16 8192^3", "kind": "gemm", "dtype": "bf16", "out": "bf16", "scales": "none", "M": 8192, "N": 8192, "K": 8192},
        # configuration 5: fp8 with fp32 scales per 128 x 128 block
        {"name": "gemm fp8 8192^3 blocks", "kind": "gemm", "dtype": "fp8", "out": "bf16", "scales": "block_f32", "M": 8192, "N": 8192, "K": 8192},
        # a prefill chunk of 1000 tokens in fp8 with the usual scaling of activations (one fp32 scale per row and 128 of k)
        {"name": "gemm fp8 1000 rows", "kind": "gemm", "dtype": "fp8", "out": "bf16", "scales": "rows_f32", "M": 1000, "N": 3584, "K": 8192},
        # the MoE layer at a decode batch, and at a prefill
        {"name": "moe f16 64 tokens", "kind": "moe", "dtype": "f16", "scales": "none", "tokens": 64},
        {"name": "moe f16 4096 tokens", "kind": "moe", "dtype": "f16", "scales": "none", "tokens": 4096},
        # the fp8 layer with fp32 scales at a prefill chunk
        {"name": "moe fp8 1024 tokens", "kind": "moe", "dtype": "fp8", "scales": "f32", "tokens": 1024},
        # configuration 2: row-major to swizzled 128 x 64 tiles
        {"name": "relayout tiles 8192^2", "kind": "relayout", "form": "tiles", "eb": 2, "rows": 8192, "cols": 8192},
        # row-major to column-major with odd extents
        {"name": "relayout transpose 8191x8193", "kind": "relayout", "form": "transpose", "eb": 2, "rows": 8191, "cols": 8193},
        # the thread map of a matrix operand held in registers (fragments, lanes, registers; copies in two waves)
        {"name": "eval operand map", "kind": "eval", "form": "operand", "rows": 2048, "cols": 4096, "given": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "moe", "relayout", "eval"])
    if kind == "gemm":
        dtype = rng.choice(["bf16", "f16", "fp8"])
        vec = 16 if dtype == "fp8" else 8                              # elements of a 16-byte chunk: what K has to be a multiple of
        M, N, K = _log(rng, 1, 4096), _log(rng, 256, 8192), _log(rng, 256, 8192)
        shape = rng.choice(["tiles", "rows", "rows", "any"])
        if shape == "tiles":
            M, N, K = -(-M // 256) * 256, -(-N // 256) * 256, -(-K // 128) * 128
        elif shape == "rows":                                          # a model's weights are round, its batch is not
            N, K = -(-N // 128) * 128, -(-K // 128) * 128
        else:
            K = -(-K // vec) * vec
        scales = rng.choice(["none", "block_f32", "rows_f32", "block_e8m0", "rows_e8m0"]) if dtype == "fp8" else "none"
        out = "f32" if rng.random() < 0.25 else ("f16" if dtype == "f16" else "bf16")
        return {"kind": kind, "dtype": dtype, "out": out, "scales": scales, "M": M, "N": N, "K": K}
    if kind == "moe":
        dtype = rng.choice(["f16", "bf16", "fp8"])
        return {"kind": kind, "dtype": dtype, "scales": rng.choice(["f32", "e8m0"]) if dtype == "fp8" else "none", "tokens": _log(rng, 1, 4096)}
    rows, cols = _log(rng, 128, 8192), _log(rng, 128, 8192)
    if kind == "relayout":
        form, eb = rng.choice(["tiles", "untile", "transpose", "pitch", "heads"]), rng.choice([1, 2, 2, 4, 8])
        if form in ("tiles", "untile"):
            rows, cols = -(-rows // 128) * 128, -(-cols // 64) * 64
        elif form == "heads":
            cols = -(-cols // 128) * 128
        while rows * cols * eb > 128 << 20:
            eb //= 2
        return {"kind": kind, "form": form, "eb": eb, "rows": rows, "cols": cols}
    form = rng.choice(["tiles", "operand"])
    rows, cols = (-(-rows // 128) * 128, -(-cols // 64) * 64) if form == "tiles" else (-(-min(rows, 4096) // 16) * 16, -(-min(cols, 4096) // 32) * 32)
    return {"kind": kind, "form": form, "rows": rows, "cols": cols, "given": rng.random() < 0.5}


# ---- inputs -------------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(g, shape, std, dtype):
    x = torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=g)
    return (x.clamp_(-448.0, 448.0) if dtype == "fp8" else x).to(TORCH[dtype])


def _scales(g, shape, dtype):
    """Scales of quantised operands: fp32 in [0.5, 2), or E8M0 codes of the powers of two 1/8 .. 8."""
    if dtype == "e8m0":
        return torch.randint(124, 131, shape, generator=g, dtype=torch.uint8, device="cuda")
    return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(0.5, 2.0, generator=g)


def _blocks(n):
    return -(-n // 128)


def _gemm_inputs(c, seed):
    """A (M, K), the image (N, K) of the column-major B, and their scales."""
    g = _gen(seed)
    M, N, K = c["M"], c["N"], c["K"]
    a = _normal(g, (M, K), 1.0, c["dtype"])
    b = _normal(g, (N, K), 1.0 if c["dtype"] == "fp8" else K ** -0.5, c["dtype"])
    sa = sb = None
    if c["scales"] != "none":
        per, st = c["scales"].split("_")
        sa = _scales(g, (M if per == "rows" else _blocks(M), _blocks(K)), st)
        sb = _scales(g, (_blocks(N), _blocks(K)), st)
    return a, b, sa, sb


def _route(g, tokens):
    """Offsets of the rows sorted by expert: every token picks TOPK distinct experts, popularities mildly unbalanced."""
    pop = torch.empty(EXPERTS, dtype=torch.float32, device="cuda").normal_(0.0, 0.5, generator=g)
    noise = torch.empty((tokens, EXPERTS), dtype=torch.float32, device="cuda").exponential_(1.0, generator=g)
    pick = (pop - noise.log()).topk(TOPK, dim=1).indices
    counts = torch.bincount(pick.reshape(-1), minlength=EXPERTS)
    return torch.cat([counts.new_zeros(1), counts.cumsum(0)]).to(torch.int32)


def _moe_inputs(c, seed):
    """Row offsets, activations, each expert's gate and up rows one after the other, down projections; in fp8 also the
    second product's quantised activations and the scales (activations, weights) of both products."""
    g = _gen(seed)
    M, dt = c["tokens"] * TOPK, c["dtype"]
    rows = _route(g, c["tokens"])
    x = _normal(g, (M, HIDDEN), 1.0, dt)
    w1 = _normal(g, (EXPERTS, 2 * INTER, HIDDEN), 1.0 if dt == "fp8" else HIDDEN ** -0.5, dt)
    w2 = _normal(g, (EXPERTS, HIDDEN, INTER), 1.0 if dt == "fp8" else INTER ** -0.5, dt)
    if dt != "fp8":
        return rows, x, w1, w2, None, None
    h = _normal(g, (M, INTER), 1.0, dt)
    # (the gate is kept where a trained one is, around one: the products of unit-variance rows are sqrt(HIDDEN) wide)
    unit = HIDDEN ** -0.5 if c["scales"] == "f32" else 1.0
    s = [_scales(g, (M, _blocks(HIDDEN)), c["scales"]), _scales(g, (EXPERTS, 2 * INTER // 128, _blocks(HIDDEN)), c["scales"]),
         _scales(g, (M, _blocks(INTER)), c["scales"]), _scales(g, (EXPERTS, HIDDEN // 128, _blocks(INTER)), c["scales"])]
    if unit != 1.0:
        s[1] = s[1] * unit
    else:
        s[1] = s[1] - 5                                                # 2^-5, the power of two nearest to 1 / sqrt(HIDDEN)
    return rows, x, w1, w2, h, s


def _interleave(w):
    """(experts, gate rows then up rows, k) -> rows of both in runs of 16, as the gated epilogue reads them."""
    E, n, k = w.shape
    return w.view(torch.uint8).reshape(E, 2, n // 32, 16, -1).transpose(1, 2).contiguous().view(w.dtype).reshape(E, n, k)


def _layouts(c):
    """(source spec, destination spec, elements of the destination buffer) of a relayout."""
    R, Cn, eb = c["rows"], c["cols"], c["eb"]
    plain = W.row_major_spec(R, Cn)
    if c["form"] in ("tiles", "untile"):
        tiles = W.blocked_swizzled_spec(R, Cn, swizzle=eb == 2)
        return (plain, tiles, R * Cn) if c["form"] == "tiles" else (tiles, plain, R * Cn)
    if c["form"] == "transpose":
        return plain, W.col_major_spec(R, Cn), R * Cn
    if c["form"] == "pitch":                                           # rows padded to whole 128-byte lines
        pitch = -(-Cn * eb // 128) * 128 // eb
        return plain, W.spec([(R, pitch, "m"), (Cn, 1, "m")]), R * pitch
    d = 128                                                            # heads: (token, head, d) -> (head, token, d)
    return plain, W.spec([(R, d, "m"), (Cn // d, R * d, "m"), (d, 1, "m")]), R * Cn


def _eval_spec(c, seed):
    """(spec, axes) of the layout; its tensor starts at an offset of its own on the first axis."""
    R, Cn = c["rows"], c["cols"]
    if c["form"] == "tiles":
        return dict(W.blocked_swizzled_spec(R, Cn), O={"m": _origin(seed)}), ["m"]
    # 16 x 32 fragments of a 16-bit MFMA operand: lane = row + 16 (k / 8), 8 consecutive k per lane, two waves hold a copy
    return W.spec([(R // 16, Cn // 32, "frag"), (16, 1, "lane"), (Cn // 32, 1, "frag"), (4, 16, "lane"), (8, 1, "reg")],
                  R=[(2, 1, "wave")], O={"frag": _origin(seed)}), ["frag", "wave", "lane", "reg"]


# ---- the calls ----------------------------------------------------------------------------------------------------

def prepare(case, seed):
    c = case
    if c["kind"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        a, b, sa, sb = _gemm_inputs(c, seed)
        desc = B.GemmDesc(M, N, K, CODE[c["dtype"]], CODE[c["out"]], B.Layout(W.row_major_spec(M, K)), B.Layout(W.col_major_spec(K, N)),
                          B.Layout(W.row_major_spec(M, N)), M * K, N * K, M * N, sa, sb,
                          scale_dtype=B.AXE_SCALE_E8M0 if c["scales"].endswith("e8m0") else B.AXE_SCALE_F32,
                          scale_a_rows=1 if c["scales"].startswith("rows") else 0)
        return {"kind": "gemm", "desc": desc, "a": a, "b": b, "c": torch.zeros((M, N), dtype=TORCH[c["out"]], device="cuda")}
    if c["kind"] == "moe":
        rows, x, w1, w2, h_in, s = _moe_inputs(c, seed)
        M, dt = x.shape[0], CODE[c["dtype"]]
        fp8 = c["dtype"] == "fp8"
        half = torch.bfloat16 if fp8 else x.dtype
        h = torch.zeros((M, INTER), dtype=half, device="cuda")
        out = torch.zeros((M, HIDDEN), dtype=half, device="cuda")
        st = B.AXE_SCALE_E8M0 if c["scales"] == "e8m0" else B.AXE_SCALE_F32
        d1 = B.GroupedGemmDesc(M, 2 * INTER, HIDDEN, EXPERTS, B.Layout(W.row_major_spec(M, HIDDEN)), B.Layout(W.gated_b_spec(HIDDEN, 2 * INTER, EXPERTS)),
                               B.Layout(W.row_major_spec(M, INTER)), M * HIDDEN, w1.numel(), M * INTER, dt, CODE["bf16"] if fp8 else dt,
                               epilogue=B.AXE_EPI_SWIGLU, scale_a=s and s[0], scale_b=s and s[1], scale_dtype=st)
        d2 = B.GroupedGemmDesc(M, HIDDEN, INTER, EXPERTS, B.Layout(W.row_major_spec(M, INTER)),
                               B.Layout(W.spec([(EXPERTS, HIDDEN * INTER, "m"), (INTER, 1, "m"), (HIDDEN, INTER, "m")])),
                               B.Layout(W.row_major_spec(M, HIDDEN)), M * INTER, w2.numel(), M * HIDDEN, dt, CODE["bf16"] if fp8 else dt,
                               scale_a=s and s[2], scale_b=s and s[3], scale_dtype=st)
        sync = None if fp8 else torch.zeros(M + 1, dtype=torch.int32, device="cuda")
        return {"kind": "moe", "fp8": fp8, "d1": d1, "d2": d2, "x": x, "w1": _interleave(w1), "w2": w2, "h_in": h_in, "h": h, "out": out,
                "rows": rows, "sync": sync, "scales": s}
    if c["kind"] == "relayout":
        src_spec, dst_spec, n = _layouts(c)
        R, Cn, eb = c["rows"], c["cols"], c["eb"]
        src = torch.randint(0, 256, (R * Cn * eb,), generator=_gen(seed), dtype=torch.uint8, device="cuda").view(WORDS[eb])
        return {"kind": "relayout", "src_l": B.Layout(src_spec), "dst_l": B.Layout(dst_spec), "shape": (R, Cn), "src": src,
                "dst": torch.zeros(n, dtype=WORDS[eb], device="cuda")}
    spec, axes = _eval_spec(c, seed)
    n = c["rows"] * c["cols"]
    layout = B.Layout(spec, axes)
    return {"kind": "eval", "layout": layout, "shape": (c["rows"], c["cols"]), "n": n, "idx": _indices(c, seed) if c["given"] else None,
            "out": torch.zeros((n, layout.E_R, len(axes)), dtype=torch.int64, device="cuda")}


def _indices(c, seed):
    n = c["rows"] * c["cols"]
    return torch.randint(0, n, (n,), generator=_gen(seed), dtype=torch.int64, device="cuda")


def _origin(seed):
    return 512 * (seed % 8191)                                         # (a multiple of the swizzle period)


def run(state):
    s = state
    if s["kind"] == "gemm":
        return B.axe_gemm(s["desc"], s["a"], s["b"], s["c"])
    if s["kind"] == "moe":
        if s["fp8"]:
            B.axe_gemm_grouped(s["d1"], s["x"], s["w1"], s["h"], s["rows"])
            B.axe_gemm_grouped(s["d2"], s["h_in"], s["w2"], s["out"], s["rows"])
        else:
            B.axe_gemm_grouped_pair(s["d1"], s["d2"], s["x"], s["w1"], s["h"], s["w2"], s["out"], s["rows"], s["sync"])
        return s["h"], s["out"]
    if s["kind"] == "relayout":
        return B.axe_relayout(s["src_l"], s["dst_l"], s["shape"], s["src"], s["dst"])
    return B.axe_layout_eval(s["layout"], s["shape"], s["n"], s["idx"], s["out"])


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    c = case
    eb = 1 if c.get("dtype") == "fp8" else 2
    if c["kind"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        bytes_ = (M * K + N * K) * eb + M * N * (4 if c["out"] == "f32" else 2)
        if c["scales"] != "none":
            bytes_ += ((M if c["scales"].startswith("rows") else _blocks(M)) + _blocks(N)) * _blocks(K) * (4 if c["scales"].endswith("f32") else 1)
        return {"bytes": bytes_, "flops": 2 * M * N * K}
    if c["kind"] == "moe":
        M = c["tokens"] * TOPK
        active = EXPERTS * (1 - (1 - TOPK / EXPERTS) ** c["tokens"])   # experts that have rows (popularities taken as equal)
        weights = active * 3 * HIDDEN * INTER * eb
        acts = M * (HIDDEN * eb + INTER * 2 + (INTER if c["dtype"] == "fp8" else 0) + HIDDEN * 2)
        return {"bytes": weights + acts, "flops": 2 * M * 3 * HIDDEN * INTER}
    n = c["rows"] * c["cols"]
    if c["kind"] == "relayout":
        return {"bytes": 2 * n * c["eb"], "flops": 0}
    return {"bytes": n * (8 * (1 if c["form"] == "tiles" else 8) + (8 if c["given"] else 0)), "flops": 0}


def tolerance(case):
    c = case
    if c["kind"] in ("relayout", "eval"):
        return "exact"
    # four times what separates a result from the one in 64 bits: the rounding of the result itself (bf16 1.7e-3, fp16
    # 2.1e-4), in the layer that of the intermediate rows and of the gate as well; results in fp32: their sums
    # (16-bit inputs up to 6e-7 at K = 8192, fp8 1.5e-5: its matrix instructions align products to the largest)
    if c["kind"] == "moe":
        return {"rel": 1.2e-3 if c["dtype"] == "f16" else 1e-2}
    if c["out"] == "f32":
        return {"rel": 6e-5 if c["dtype"] == "fp8" else 2.4e-6}
    return {"rel": 8.5e-4 if c["out"] == "f16" else 6.7e-3}


# ---- the same in 64 bits, in plain torch ---------------------------------------------------------------------------

def _f64(x):
    return (x.to(torch.float32) if x.dtype == torch.float8_e4m3fn else x).double()


def _scale64(s):
    return torch.exp2(s.double() - 127.0) if s.dtype == torch.uint8 else s.double()


def _dequantised(x, s, rows):
    """x (R, K) times its scales (ceil(R / rows), ceil(K / 128))."""
    x = _f64(x)
    if s is None:
        return x
    s = _scale64(s).repeat_interleave(128, 1)[:, :x.shape[1]]
    return x * (s if rows == 1 else s.repeat_interleave(rows, 0)[:x.shape[0]])


def exact(case, seed):
    c = case
    if c["kind"] == "gemm":
        a, b, sa, sb = _gemm_inputs(c, seed)
        return _dequantised(a, sa, 1 if c["scales"].startswith("rows") else 128) @ _dequantised(b, sb, 128).t()
    if c["kind"] == "moe":
        rows, x, w1, w2, h_in, s = _moe_inputs(c, seed)
        s = s or [None] * 4
        at = rows.tolist()
        h = torch.zeros((x.shape[0], INTER), dtype=torch.float64, device="cuda")
        out = torch.zeros((x.shape[0], HIDDEN), dtype=torch.float64, device="cuda")
        cut = lambda t, i, j: None if t is None else t[i:j]            # noqa: E731
        for e in range(EXPERTS):
            i, j = at[e], at[e + 1]
            if i == j:
                continue
            p = _dequantised(x[i:j], cut(s[0], i, j), 1) @ _dequantised(w1[e], None if s[1] is None else s[1][e], 128).t()
            gate, up = p[:, :INTER], p[:, INTER:]
            h[i:j] = gate / (1.0 + torch.exp(-gate)) * up
            left = h[i:j] if h_in is None else _dequantised(h_in[i:j], cut(s[2], i, j), 1)
            out[i:j] = left @ _dequantised(w2[e], None if s[3] is None else s[3][e], 128).t()
        return h, out
    R, Cn = c["rows"], c["cols"]
    if c["kind"] == "relayout":
        eb = c["eb"]
        src = torch.randint(0, 256, (R * Cn * eb,), generator=_gen(seed), dtype=torch.uint8, device="cuda").view(WORDS[eb])
        if c["form"] == "tiles":
            return _swizzled(src.reshape(R // 128, 128, Cn // 64, 64).transpose(1, 2), eb).reshape(-1)
        if c["form"] == "untile":
            return _swizzled(src.reshape(R // 128, Cn // 64, 128, 64), eb).transpose(1, 2).reshape(-1)
        if c["form"] == "transpose":
            return src.reshape(R, Cn).t().reshape(-1)
        if c["form"] == "pitch":
            pitch = -(-Cn * eb // 128) * 128 // eb
            dst = torch.zeros((R, pitch), dtype=WORDS[eb], device="cuda")
            dst[:, :Cn] = src.reshape(R, Cn)
            return dst.reshape(-1)
        return src.reshape(R, Cn // 128, 128).transpose(0, 1).reshape(-1)
    n = R * Cn
    i = _indices(c, seed) if c["given"] else torch.arange(n, device="cuda")
    r, k = i // Cn, i % Cn
    if c["form"] == "tiles":
        m = (r // 128) * (Cn // 64) * 8192 + (k // 64) * 8192 + (r % 128) * 64 + k % 64 + _origin(seed)
        return (m ^ (((m >> 6) & 7) << 3)).reshape(n, 1, 1)
    out = torch.empty((n, 2, 4), dtype=torch.int64, device="cuda")
    out[:, :, 0] = ((r // 16) * (Cn // 32) + k // 32 + _origin(seed))[:, None]
    out[:, :, 1] = torch.arange(2, device="cuda")
    out[:, :, 2] = (r % 16 + 16 * (k // 8 % 4))[:, None]
    out[:, :, 3] = (k % 8)[:, None]
    return out


def _swizzled(t, eb):
    """(.., .., 128, 64) tiles with the eight 16-byte chunks of each row exchanged by row mod 8 (2-byte elements only)."""
    if eb != 2:
        return t
    t = t.reshape(*t.shape[:2], 16, 8, 8, 8)                           # row / 8, row % 8, chunk, element
    key = torch.arange(8, device=t.device)[:, None] ^ torch.arange(8, device=t.device)[None, :]
    return t.gather(4, key[None, None, None, :, :, None].expand(t.shape)).reshape(*t.shape[:2], 128, 64)
