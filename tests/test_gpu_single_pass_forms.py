"""The two forms of the single-pass compress (one workgroup per token; persistent workgroups) at the shapes where they
can go wrong: both sides of the line between them, edges of the placement's blocks of 2048 tokens, the last run
of a row cut short, tokens with more outliers than a wave keeps in LDS.  Whole blobs against the oracle."""
import numpy as np
import pytest

from paper_2511_04002_amd import synth
from test_gpu_parity import check_parity, tsq  # noqa: F401

pytestmark = pytest.mark.gpu


def rows(T, H, dtype, heavy=0):
    g = np.random.Generator(np.random.PCG64(T * 7 + H))
    v = g.standard_normal((T, H)) * g.lognormal(0.0, 0.8, (T, 1))
    v[g.random((T, H)) < 0.004] *= 30.0
    for i, t in enumerate(g.choice(T, heavy, replace=False)):
        n = (H // 10, H // 8, H // 4, H // 2, H)[i % 5]
        v[t, g.choice(H, n, replace=False)] = 50.0 * g.choice([-1.0, 1.0], n)
    return synth.to_f16_bits(v) if dtype == "f16" else synth.to_bf16_bits(v)


# tokens * waves <= 8192: one workgroup per token (rows of one wave: always)
@pytest.mark.parametrize("T,H,dtype", [(2047, 72, "f16"), (2048, 72, "bf16"), (2049, 72, "f16"), (6145, 1000, "bf16"),
                                       (3072, 4096, "f16"), (3073, 4088, "bf16"), (2048, 5120, "bf16"), (2049, 6144, "f16"),
                                       (1536, 8192, "bf16"), (1537, 8192, "f16"), (385, 16384, "f16"), (769, 8200, "bf16"),
                                       (100, 32768, "bf16"), (4096, 4096, "f16"), (4097, 2056, "bf16"), (2730, 5120, "f16"),
                                       (2731, 6144, "bf16"), (512, 32768, "f16"), (513, 16400, "bf16")])
def test_both_sides_of_the_line_and_block_edges(tsq, oracle, T, H, dtype):
    check_parity(tsq, oracle, rows(T, H, dtype), dtype, 6.0, (2, 3, 4, 6, 8), 0.1, "rel_rms", "fused", label="T=%d H=%d" % (T, H))


@pytest.mark.parametrize("T,H,dtype", [(40, 4096, "f16"), (40, 1032, "bf16"), (3200, 4096, "f16"), (1600, 8192, "bf16")])
def test_tokens_full_of_outliers(tsq, oracle, T, H, dtype):
    ref, _ = check_parity(tsq, oracle, rows(T, H, dtype, heavy=30), dtype, 6.0, (2, 4, 8), 0.05, "rel_rms", "fused",
                          label="heavy rows T=%d H=%d" % (T, H))
    assert np.diff(ref.row_ptr.astype(np.int64)).max() == H
