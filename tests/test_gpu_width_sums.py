"""The sums over a workgroup behind Algorithm 1's test, at every largest width and number of waves.  Whole blobs against
the oracle."""
import pytest

from test_gpu_parity import check_parity, tsq  # noqa: F401
from test_gpu_single_pass_forms import rows

pytestmark = pytest.mark.gpu


# the sum behind the test counts lowest bits that differ between the shifted reference and the candidate: every pair of
# widths, in workgroups of every number of waves, with budgets that let the search go on to the narrow ones
@pytest.mark.parametrize("bits", [(3, 2), (4, 3, 2), (5, 4, 3, 2), (6, 5, 4, 3, 2), (7, 6, 5, 4, 3, 2), (8, 7, 6, 5, 4, 3, 2), (8, 2), (7, 3)])
@pytest.mark.parametrize("T,H,dtype", [(60, 2048, "bf16"), (50, 4096, "f16"), (40, 5128, "bf16"), (30, 8192, "f16"),
                                       (20, 16384, "bf16"), (10, 32768, "f16")])
def test_sums_at_every_pair_of_widths(tsq, oracle, bits, T, H, dtype):
    for eps, mode in ((0.1, "rel_rms"), (0.4, "rel_rms"), (0.45, "lsb")):
        check_parity(tsq, oracle, rows(T, H, dtype), dtype, 6.0, bits, eps, mode, "fused", label="%s eps=%g" % (bits, eps))
