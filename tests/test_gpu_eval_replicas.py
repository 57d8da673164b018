"""Layout evaluation with replicas or many axes (the kernel that writes an index's words as consecutive pairs) against the
oracle: every number of axes, odd and even words per index, 256 words and one index more than that allows, given indices
inside and outside the layout, tails of a workgroup, a swizzle on top of replicas, negative strides."""
import numpy as np
import pytest
import torch

from oracle import axe_ref as R
from oracle.axe_layout import Layout
from paper_2601_19092_amd import binding as B
from paper_2601_19092_amd import workloads as W

pytestmark = pytest.mark.gpu
I64MIN = np.iinfo(np.int64).min


def case(naxes, replicas, swizzle=None):
    axes = [f"x{a}" for a in range(naxes)]
    D = [(7, 320, axes[0]), (4, 64, axes[-1]), (5, -3, axes[naxes // 2]), (8, 8, axes[0]), (3, 1, axes[-1])]
    Rp = [(e, s, axes[i % naxes]) for i, (e, s) in enumerate(replicas)]
    O = {axes[0]: 1024, axes[naxes // 2]: 17} if naxes > 1 else {axes[0]: 1024}
    return W.spec(D, R=Rp, O=O, swizzle=swizzle), axes, 7 * 4 * 5 * 8 * 3


@pytest.mark.parametrize("naxes,replicas", [(1, [(2, 4096)]), (1, [(3, 4096), (85, 8192)]), (2, [(3, 1)]), (3, []), (4, [(2, 1)]), (4, [(64, 1)]),
                                            (5, []), (5, [(3, 2)]), (6, [(2, -1), (3, 5)]), (7, [(5, 1)]), (7, [(36, 1)]), (8, [(32, 1)]), (8, [(33, 1)]),
                                            (1, [(256, 4096)]), (1, [(257, 4096)])])
@pytest.mark.parametrize("given", [False, True])
def test_eval_matches_the_oracle(naxes, replicas, given):
    spec, axes, E = case(naxes, replicas, ("x0", 3, 3, 6) if naxes != 3 else None)
    L, Lo = B.Layout(spec, axes), Layout.from_spec(spec)
    shape = (E // 24, 24)
    for n in (E, 256, 257, 1, 511):
        idx = np.random.default_rng(n).integers(0, E, n) if given else np.arange(n)
        want = R.evaluate_np(Lo, idx, axes)
        d_idx = None
        if given:
            asked = idx.copy()
            asked[::5] = [(-1, E, -2 ** 40, E + 2 ** 33)[i % 4] for i in range(len(asked[::5]))]
            want[::5] = I64MIN
            d_idx = torch.from_numpy(asked).cuda()
        guard = torch.full((n * L.E_R * naxes + 2,), 77, dtype=torch.int64, device="cuda")
        out = guard[:-2].view(n, L.E_R, naxes)
        B.axe_layout_eval(L, shape, n, d_idx, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want), n
        assert (guard[-2:] == 77).all(), "written past the end"
        odd = torch.zeros(n * L.E_R * naxes + 1, dtype=torch.int64, device="cuda")[1:].view(n, L.E_R, naxes)   # 8 bytes off a pair
        B.axe_layout_eval(L, shape, n, d_idx, odd)
        assert torch.equal(odd, out)


@pytest.mark.parametrize("extents", [(3, 7, 11, 13), (2147483647,), (46341, 46339), (1073741825, 1), (2, 1073741823), (5, 3, 715827, 199), (65537, 32765)])
def test_eval_divides_exactly_by_any_extent(extents):
    """Digits come from multiplications: extents around powers of two, primes, index spaces up to 2^31 - 1, at the indices where
    a quotient steps."""
    D, s = [], 1
    for e in reversed(extents):
        D.insert(0, (e, s, "m"))
        s *= e + 1                                             # the digits stay readable in the coordinate
    L, Lo = B.Layout(W.spec(D)), Layout.from_spec(W.spec(D))
    E = int(np.prod([int(e) for e in extents], dtype=object))
    last = int(extents[-1])
    rng = np.random.default_rng(1)
    q = rng.integers(0, max(1, E // last), 4000)
    idx = np.unique(np.clip(np.concatenate([q * last - 1, q * last, q * last + 1, rng.integers(0, E, 4000), [0, E - 1, E - 2, E // 2]]), 0, E - 1))
    got = B.axe_layout_eval(L, (E,), len(idx), torch.from_numpy(idx).cuda()).cpu().numpy()
    assert np.array_equal(got, R.evaluate_np(Lo, idx, ["m"]))
