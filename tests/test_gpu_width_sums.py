"""The sums over a workgroup behind Algorithm 1's test, at every largest width and number of waves, in workgroups of one
token and of several.  Whole blobs against the oracle."""
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
    reached = set()
    for eps, mode in ((0.1, "rel_rms"), (0.4, "rel_rms"), (0.45, "lsb")):
        ref, _ = check_parity(tsq, oracle, rows(T, H, dtype), dtype, 6.0, bits, eps, mode, "fused", label="%s eps=%g" % (bits, eps))
        reached |= set(ref.bits.tolist())
    assert min(bits) in reached                              # some token's search went all the way down


PAIRS = [(a, b) for a in range(3, 9) for b in range(2, a)]


# two widths and a budget at which half of the tokens fail: the sum itself decides, token by token
@pytest.mark.parametrize("T,H,dtype,tokens_per_workgroup", [
    (64, 2048, "f16", 1), (64, 2600, "bf16", 1), (64, 6144, "f16", 1), (64, 8192, "bf16", 1), (32, 16384, "f16", 1), (32, 32768, "bf16", 1),
    (1027, 2048, "bf16", 8), (1025, 4096, "f16", 2), (1283, 2856, "bf16", 2), (2305, 6152, "f16", None)])
def test_the_sum_decides_at_every_pair_of_widths(tsq, oracle, T, H, dtype, tokens_per_workgroup):
    x = rows(T, H, dtype)
    plan = tsq.Plan(T, H, dtype, 6.0, (2, 8), 0.1, pipeline="fused").handle
    if tokens_per_workgroup is None:
        assert tsq.tsq_plan_kernel(plan) == "k_fused"
    else:
        assert tsq.tsq_plan_direct_launch(plan)[0] == tokens_per_workgroup
    for bits in PAIRS if T < 1000 else PAIRS[::3] + [(8, 2)]:
        lo, hi = 0.0, 2.0
        for _ in range(12):
            eps = 0.5 * (lo + hi)
            r = oracle.compress(x[:48], oracle.F16 if dtype == "f16" else oracle.BF16, 6.0, bits, eps, 1, nthreads=8)
            lo, hi = (lo, eps) if (r.bits == bits[1]).mean() > 0.5 else (eps, hi)
        ref, _ = check_parity(tsq, oracle, x, dtype, 6.0, bits, eps, "rel_rms", "fused", label="%s eps=%g" % (bits, eps))
        assert set(ref.bits.tolist()) == set(bits)
