"""Restore of every width: codes taken apart four at a time, signs put in behind the conversion to 16 bits.  Rows whose restored
values are subnormal, of ordinary size and close to the type's largest; rows that end inside a run and inside four codes' word."""
import numpy as np
import pytest

from paper_2511_04002_amd import synth
from test_gpu_rans import tsq  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("b", [2, 3, 4, 5, 6, 7, 8])
def test_restored_bits_of_every_width(tsq, oracle, dtype, b):
    import torch
    for H in (8, 40, 2056, 4096 + 24):
        g = np.random.Generator(np.random.PCG64(1000 * b + H))
        scale = np.repeat([6e-8, 3e-6, 1.0, 3e4], 5)[:, None]
        v = np.clip(g.standard_normal((20, H)), -2.0, 2.0) * scale
        v[:, 0] = 2.0 * scale[:, 0]
        v[4] = 0.0
        x = synth.to_f16_bits(v) if dtype == "f16" else synth.to_bf16_bits(v)
        dt = {"f16": 0, "bf16": 1}[dtype]
        ref = oracle.compress(x, dt, 65000.0, (b,), 0.05, 1, nthreads=4)
        plan = tsq.Plan(20, H, dtype, 65000.0, (b,), 0.05, max_outliers=64)
        blob = plan.compress(torch.from_numpy(x.view(np.int16)).cuda())
        assert plan.info(blob).status == 0
        got = plan.decompress(blob).cpu().numpy().view(np.uint16)
        assert np.array_equal(got, oracle.decompress(ref)), (dtype, b, H)
