"""Restore of every width: codes taken apart four at a time, signs put in behind the conversion to 16 bits.  Rows whose restored
values are zeros (a code of magnitude 0 has no sign), of ordinary size and close to the type's largest, for fp16 also subnormal ones
(bfloat16 rows have none: a row whose largest magnitude is below 2^-100 is restored as zeros); rows that end inside a run and inside four
codes' word."""
import numpy as np
import pytest

from paper_2511_04002_amd import synth
from test_gpu_rans import tsq  # noqa: F401

pytestmark = pytest.mark.gpu

# dtype -> magnitudes of the rows (half of the largest element), tau, smallest normal and a large pattern
ROWS = {"f16": ((6e-8, 3e-6, 1.0, 3e4), 65000.0, 0x0400, 0x7B00),
        "bf16": ((1e-40, 2.0 ** -100, 1.0, 1.6e38), 3.38e38, 0x0080, 0x7F40)}


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("b", [2, 3, 4, 5, 6, 7, 8])
def test_restored_bits_of_every_width(tsq, oracle, dtype, b):
    import torch
    scales, tau, normal, large = ROWS[dtype]
    seen = []
    for H in (8, 40, 2056, 4096 + 24):
        g = np.random.Generator(np.random.PCG64(1000 * b + H))
        scale = np.repeat(scales, 5)[:, None]
        v = np.clip(g.standard_normal((20, H)), -2.0, 2.0) * scale
        v[:, 0] = 2.0 * scale[:, 0]
        v[4] = 0.0
        x = synth.to_f16_bits(v) if dtype == "f16" else synth.to_bf16_bits(v)
        dt = {"f16": 0, "bf16": 1}[dtype]
        ref = oracle.compress(x, dt, tau, (b,), 0.05, 1, nthreads=4)
        assert ref.nnz == 0
        want = oracle.decompress(ref)
        plan = tsq.Plan(20, H, dtype, tau, (b,), 0.05, max_outliers=64)
        blob = plan.compress(torch.from_numpy(x.view(np.int16)).cuda())
        assert plan.info(blob).status == 0
        got = plan.decompress(blob).cpu().numpy().view(np.uint16)
        assert np.array_equal(got, want), (dtype, b, H)
        seen.append(want.ravel())
    seen = np.concatenate(seen)
    magnitude = seen & 0x7FFF
    assert (seen == 0).any() and not (seen == 0x8000).any()
    assert (magnitude >= large).any() and (seen >= 0x8000 + large).any()
    if dtype == "f16":
        below = (magnitude > 0) & (magnitude < normal)
        assert below.any() and (below & (seen >= 0x8000)).any()
