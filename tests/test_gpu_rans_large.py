"""The entropy stage where the codes are more than the caches hold (another form of the decoder's stores): the payload comes back."""
import pytest

from test_gpu_rans import tsq  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H", [(24577, 4096), (34000, 2968)])        # 96 MiB and one row's codes; rows that end inside a run
def test_codes_past_the_caches_come_back(tsq, T, H):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T)
    x = torch.randn((T, H), device="cuda", generator=gen) * torch.exp(0.5 * torch.randn((T, 1), device="cuda", generator=gen))
    plan = tsq.Plan(T, H, "f16", 8.0, (2, 3, 4, 5, 6, 7, 8), 0.08, max_outliers=T * H // 4)
    assert plan.layout.payload_capacity > 96 << 20
    blob = plan.compress(x.half().view(torch.int16))
    info = plan.info(blob)
    at, n = int(plan.layout.off_payload), int(info.payload_bytes)
    want = blob[at: at + n].clone()
    eblob = plan.entropy_encode(blob)
    blob[at: at + n] = 0xEE
    plan.entropy_decode(eblob, blob)
    assert torch.equal(blob[at: at + n], want)
