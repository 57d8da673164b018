"""The fused pair on tiles of 192 rows: edges of its tiles and fragments against the oracle and, bit for bit, against two launches on tiles of 128 rows and
against the checking build."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2601_19092_amd import binding as B
from test_gpu_grouped_pair import TOL, Layer, check_blocks, decode, run_pair
from test_gpu_paranoid_build import PARANOID, library

pytestmark = pytest.mark.gpu

# Sizes that average between 208 and 288 rows: what few groups take 192 rows for.  (sizes, hidden, intermediate, out): the smallest K on both sides;
# one row block more or less a row; fragments of 16 rows, a wave's half of 96.
CASES = [([191, 192, 193, 384, 385, 0, 1, 500], 256, 256, 256), ([95, 96, 97, 577, 15, 17, 700, 288, 480], 512, 384, 512)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_pair_on_192_rows(case, dtype):
    sizes, hidden, inter, out = CASES[case]
    assert 208 * len(sizes) < sum(sizes) <= 288 * len(sizes)
    L = Layer(list(np.concatenate([[0], np.cumsum(sizes)])), hidden, inter, out, 900 + case, dtype)
    assert B.axe_gemm_grouped_pair_fused(*L.descs(B.AXE_GROUPED_AUTO))
    h, c, _ = run_pair(L, B.AXE_GROUPED_AUTO)
    h_ref, c_ref = L.oracle()
    check_blocks(L.off, decode(h, dtype), h, h_ref, TOL[dtype], "H")
    check_blocks(L.off, decode(c, dtype), c, c_ref, TOL[dtype], "C")
    for h2, c2, _ in (run_pair(L, B.AXE_GROUPED_TILES_128, fused=False), run_pair(L, B.AXE_GROUPED_TILES_256)):
        assert np.array_equal(h, h2) and np.array_equal(c, c2)
    with library(PARANOID):
        h2, c2, _ = run_pair(L, B.AXE_GROUPED_AUTO)
    assert np.array_equal(h, h2) and np.array_equal(c, c2)
