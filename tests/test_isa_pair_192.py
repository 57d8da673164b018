"""The fused pair on tiles of 192 rows, on the ISA hipcc emits: what the pairs on the other heights are checked for."""
import pytest

from test_isa_invariants import isa, test_fused_pair_publishes_with_write_through_stores_and_acquires_before_it_reads as check  # noqa: F401


@pytest.mark.parametrize("kernel", ["gemm_bf16_192_grouped_pair_kernel", "gemm_f16_192_grouped_pair_kernel"])
def test_pair_on_192_rows(isa, kernel):  # noqa: F811
    check(isa, kernel)
