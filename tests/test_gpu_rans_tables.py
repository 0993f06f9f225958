"""The encode call's tables where the counting workgroups' sets are added up by one workgroup per width class or by several
(64 sets each, a set per 16 tokens or more), and its streams where their words end inside a 16-byte piece."""
import numpy as np
import pytest

from paper_2511_04002_amd import synth
from test_gpu_rans import RE, check, tsq  # noqa: F401

pytestmark = pytest.mark.gpu


# one slice of sets up to 1024 tokens; then two, and eight from 7169 on; more than 512 sets' worth: sets of 17 tokens
@pytest.mark.parametrize("T", [1, 17, 1024, 1025, 2049, 7168, 7169, 8193])
def test_tables_of_one_and_of_several_slices(tsq, oracle, RE, T):
    import torch
    R, E = RE
    H = 16
    g = np.random.Generator(np.random.PCG64(100 + T))
    # loud and quiet tokens: every width occurs, some codes once (frequencies that had to be raised to 1 and cut elsewhere)
    v = g.standard_t(3, size=(T, H)) * g.lognormal(0.0, 1.0, (T, 1))
    x = synth.to_bf16_bits(v)
    widths = (2, 3, 4, 5, 6, 7, 8)
    ref = oracle.compress(x, 1, 10.0, widths, 0.1, 1, nthreads=8)
    plan = tsq.Plan(T, H, "bf16", 10.0, widths, 0.1, max_outliers=max(ref.nnz, 1))
    blob = plan.compress(torch.from_numpy(x.view(np.int16)).cuda())
    eblob, ews = plan.new_entropy_blob(), plan.new_entropy_workspace()
    ews.fill_(0xA5)
    want = R.class_tables(E.code_histogram(ref), ref.bits)
    for _ in range(2):                                   # (the workspace as the first call left it)
        plan.entropy_encode(blob, eblob, ews)
        assert np.array_equal(plan.entropy_sections(eblob)["tables"], want)
    blob2 = blob.clone()
    at = int(plan.layout.off_payload)
    blob2[at: at + int(plan.layout.payload_capacity)] = 0xEE
    plan.entropy_decode(eblob, blob2)
    assert np.array_equal(plan.sections(blob2)["payload"], ref.payload)


@pytest.mark.parametrize("H", [64, 72, 80, 88, 8192 + 8])
def test_streams_that_end_inside_a_piece(tsq, oracle, RE, H):
    """Forty tokens of noise: numbers of words that eight does not divide, odd ones among them, in streams of less and of more than the 6 KB
    that move before their place is known."""
    g = np.random.Generator(np.random.PCG64(H))
    v = np.clip(g.standard_normal((40, H)) * 2.0, -5.5, 5.5) * g.uniform(0.2, 1.0, (40, 1))
    check(tsq, oracle, RE, synth.to_f16_bits(v), "f16", 6.0, (8,), 0.05, label="pieces H=%d" % H)
