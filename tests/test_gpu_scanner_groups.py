"""The persistent compress kernel's placement at the token counts where its scanner can go wrong (a lane takes four tokens,
a group 256, a round 1024).  Whole blobs against the oracle."""
import pytest

from test_gpu_parity import check_parity, tsq  # noqa: F401
from test_gpu_single_pass_forms import kernel_of, rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,dtype", [(4097, 4096, "f16"), (4354, 2056, "bf16"), (5119, 2504, "f16"), (5120, 4088, "bf16"),
                                       (5123, 4096, "f16"), (2816, 5120, "bf16"), (3071, 6144, "f16"), (3074, 4104, "bf16"),
                                       (2303, 8192, "f16"), (2305, 6152, "bf16"), (1282, 8200, "f16"), (1025, 16384, "bf16"),
                                       (514, 32768, "f16")])
def test_token_counts_around_the_scanner_s_groups(tsq, oracle, T, H, dtype):
    assert kernel_of(tsq, T, H, dtype) == "k_fused"
    check_parity(tsq, oracle, rows(T, H, dtype), dtype, 6.0, (2, 4, 8), 0.1, "rel_rms", "fused", label="T=%d H=%d" % (T, H))
