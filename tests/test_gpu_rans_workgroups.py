"""The decoder's workgroups (512 at most, sixteen tokens at a time, a table each for the three most frequent width
classes, ranks and a list for the others) at the token counts and row
lengths where they can go wrong: fewer tokens than workgroups, one more than they take in a turn, more width
classes among a workgroup's tokens than it has tables for, lanes beyond the row, rows that end inside a run, streams that
go round a wave's ring of words.  Tables, offsets, streams and the restored payload against the oracle, byte for byte."""
import numpy as np
import pytest

from paper_2511_04002_amd import synth
from test_gpu_rans import RE, check, tsq  # noqa: F401

pytestmark = pytest.mark.gpu


def rows(T, H, dtype):
    """One element between 1.7 and 430 times as loud as the rest: the louder, the wider the codes, so that
    all widths are chosen."""
    g = np.random.Generator(np.random.PCG64(T * 31 + H))
    v = g.standard_normal((T, H)) * 0.3
    v[:, 0] = 2.0 ** g.uniform(-1, 7, T)
    return synth.to_f16_bits(v) if dtype == "f16" else synth.to_bf16_bits(v)


# per workgroup ceil(T / 512) tokens
@pytest.mark.parametrize("T,H,dtype", [(1, 8, "f16"), (2, 2048, "bf16"), (511, 40, "f16"), (513, 64, "bf16"),
                                           (8193, 24, "f16"), (8200, 96, "bf16"), (530, 2056, "f16"),
                                           (40, 5120, "bf16"), (3, 16384 + 24, "f16")])
def test_workgroups_of_the_decoder(tsq, oracle, RE, T, H, dtype):
    ref, _ = check(tsq, oracle, RE, rows(T, H, dtype), dtype, 1000.0, (2, 3, 4, 5, 6, 7, 8), 0.05, label="T=%d" % T)
    if T > 8192:
        per = -(-T // 512)
        classes = [len(set(ref.bits[i:i + per].tolist())) for i in range(0, T, per)]
        assert max(classes) > 4, "workgroups with classes beyond the third are among them"
