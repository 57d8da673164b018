"""E8M0 codes over their whole range 1 .. 254 on every member of the tile family: the two codes of a block may add up to a power
of two that no float holds, where the block's product is zero or so small that the result is an ordinary number."""
import numpy as np
import pytest
import torch

from paper_2601_19092_amd import binding as B
from test_tile_family import MEMBERS, descriptor, forced


def operands(M, N, K, rows, seed, kinds):
    """Codes of A and of B (one per row of A or per 128 x 128 block) and fp8 bytes; the k blocks of 128 take the kinds in turn:
    0: zeros in A under codes 254 and 254;  1: one product of the two least numbers, 2^-18, under codes that add up to 2^(128 .. 140);
    2: ordinary numbers under codes that add up to 2^-20 .. 2^20;  3: zeros in B under 254 and 250;  4: the least numbers under 1 and 1."""
    rng = np.random.default_rng(seed)
    nb = -(-K // 128)
    a, b = rng.integers(0x30, 0x40, (M, K)).astype(np.uint8), rng.integers(0x30, 0x40, (N, K)).astype(np.uint8)
    ra, rb = M if rows == 1 else -(-M // 128), -(-N // 128)
    ca, cb = np.full((ra, nb), 127, np.uint8), np.full((rb, nb), 127, np.uint8)
    for k in range(nb):
        blk = slice(128 * k, 128 * k + 128)
        if kinds[k % len(kinds)] == 0:
            a[:, blk], ca[:, k], cb[:, k] = 0, 254, 254
        elif kinds[k % len(kinds)] == 1:
            a[:, blk], b[:, blk] = 0, 0
            a[:, 128 * k], b[:, 128 * k] = 1, 1
            ca[:, k], cb[:, k] = 250, rng.integers(132, 145, rb)
        elif kinds[k % len(kinds)] == 2:
            ca[:, k], cb[:, k] = rng.integers(117, 138, ra), rng.integers(117, 138, rb)
        elif kinds[k % len(kinds)] == 3:
            b[:, blk], ca[:, k], cb[:, k] = 0, 254, 250
        else:
            a[:, blk], b[:, blk], ca[:, k], cb[:, k] = 1, 1, 1, 1
    return a, b, ca, cb


def exact(a, b, ca, cb, rows):
    val = lambda x: torch.from_numpy(x).view(torch.float8_e4m3fn).to(torch.float64).numpy()   # noqa: E731
    A, Bm, out = val(a), val(b), 0.0
    for k in range(ca.shape[1]):
        blk = slice(128 * k, 128 * k + 128)
        sa = np.exp2(ca[:, k].astype(np.float64) - 127)
        sa = sa if rows == 1 else np.repeat(sa, 128)[:a.shape[0]]
        sb = np.repeat(np.exp2(cb[:, k].astype(np.float64) - 127), 128)[:b.shape[0]]
        out = out + (A[:, blk] @ Bm[:, blk].T) * sa[:, None] * sb[None, :]
    return out


def run(d, a, b, M, N, member=None):
    dA, dB = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    dC = torch.full((M, N), -7.0, dtype=torch.float32, device="cuda")
    if member is None:
        B.axe_gemm(d, dA, dB, dC)
    else:
        with forced(member):
            assert B.axe_gemm_describe(d, B.AXE_DESC_C_STORE)[1] == MEMBERS[member][:2]
            B.axe_gemm(d, dA, dB, dC)
    torch.cuda.synchronize()
    return dC.cpu().numpy().astype(np.float64)


@pytest.mark.gpu
@pytest.mark.parametrize("member", range(len(MEMBERS)))
@pytest.mark.parametrize("rows", [0, 1])
@pytest.mark.parametrize("K,kinds", [(128 * 13, (0, 2, 3, 4)), (128 * 5 + 16, (2, 3, 0)), (128 * 9, (1, 0, 3, 4, 2)), (128 * 15, (2,) * 6 + (3, 0))])
def test_codes_of_the_whole_range(member, rows, K, kinds):
    M, N = MEMBERS[member][0] + 3, MEMBERS[member][1] + 5
    a, b, ca, cb = operands(M, N, K, rows, member, kinds)
    sa, sb = torch.from_numpy(ca).cuda(), torch.from_numpy(cb).cuda()
    got = run(descriptor(M, N, K, "fp8", "f32", (sa, sb), rows), a, b, M, N, member)
    want = exact(a, b, ca, cb, rows)
    assert np.isfinite(want).all() and np.abs(want).max() < 2.0 ** 127
    # sums in 32 bits of blocks that are exact (powers of two, or products of numbers with 4 bits): one rounding per block
    err = np.abs(got - want) / np.abs(want)
    assert err.max() <= ca.shape[1] * 2.0 ** -24


@pytest.mark.gpu
def test_the_large_tile_agrees():
    """The same codes on the 256 x 256 kernel, which had served these sizes before the family did (16-bit results: finite ones only)."""
    M, N, K = 512, 256, 128 * 13
    for rows in (0, 1):
        a, b, ca, cb = operands(M, N, K, rows, 3, (0, 2, 3, 4))
        sa, sb = torch.from_numpy(ca).cuda(), torch.from_numpy(cb).cuda()
        out = []
        for tile in (B.AXE_TILE_256x256x64, B.AXE_TILE_AUTO):
            d = descriptor(M, N, K, "fp8", "bf16", (sa, sb), rows)
            d.c.tile_hint = tile
            dC = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
            B.axe_gemm(d, torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), dC)
            out.append(dC.float().cpu().numpy())
        assert np.isfinite(out[0]).all() and np.abs(out[0] - out[1]).max() <= 2.0 ** -8 * np.abs(out[0]).max()
