"""Decoding classes whose only code has the whole frequency range (4096, which a table's word cannot hold): rows of zeros, which
are the only ones of their width, alone, as the most frequent class of a workgroup and as one of its rarest."""
import numpy as np
import pytest

from paper_2511_04002_amd import synth
from test_gpu_rans import RE, check, tsq  # noqa: F401

pytestmark = pytest.mark.gpu

WIDTHS = (2, 3, 4, 5, 6, 7, 8)


@pytest.mark.parametrize("T,H,every,budget", [(3, 8, 1, 0.05), (33, 2056, 1, 0.05), (700, 72, 2, 0.1), (8200, 40, 1.33, 0.05),
                                              (8200, 32, 17, 0.05)])
def test_rows_of_zeros_have_a_class_of_one_code(tsq, oracle, RE, T, H, every, budget):
    g = np.random.Generator(np.random.PCG64(T * 31 + H))
    v = g.standard_normal((T, H)) * 0.3
    v[:, 0] = 2.0 ** g.uniform(-1, 2.2, T)               # two louder elements: widths 4 to 7
    v[:, 1] = v[:, 0] * 0.6
    x = synth.to_f16_bits(v)
    x[np.arange(T) % every < 1] = 0
    x[oracle.compress(x, 0, 1000.0, WIDTHS, budget, 1, nthreads=8).bits == 2] = 0
    ref, _ = check(tsq, oracle, RE, x, "f16", 1000.0, WIDTHS, budget, label="zeros T=%d" % T)
    R, E = RE
    assert R.class_tables(E.code_histogram(ref), ref.bits)[0][0] == 4096
    if T > 8192:                                         # 17 tokens a workgroup: the class's place among the classes
        share = (ref.bits == 2).mean()
        assert len(set(ref.bits.tolist())) > 3 and (share > 0.7 if every < 2 else share < 0.1)
