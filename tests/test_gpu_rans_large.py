"""The entropy stage where the codes are about what the caches hold, or more: the decoder stores them in another form when
the blob holds more than 160 MB of them, whatever the plan has room for.  The payload comes back."""
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


# one width, so the codes' bytes are known: the most that takes the ordinary stores, the first that takes the other form, rows that
# end inside a run, and rows of which a wave has a second round
@pytest.mark.parametrize("T,H,past", [(40960, 4096, False), (40961, 4096, True), (56530, 2968, True), (64528, 2600, True)])
def test_codes_around_the_line_come_back(tsq, T, H, past):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H)
    x = torch.randn((T, H), device="cuda", generator=gen).half()
    plan = tsq.Plan(T, H, "f16", 8.0, (8,), 0.05, max_outliers=1024)
    blob = plan.compress(x.view(torch.int16))
    info = plan.info(blob)
    assert info.payload_bytes == T * H and (info.payload_bytes > 160 << 20) == past
    at = int(plan.layout.off_payload)
    want = blob[at: at + T * H].clone()
    eblob = plan.entropy_encode(blob)
    blob[at: at + T * H] = 0xEE
    plan.entropy_decode(eblob, blob)
    assert torch.equal(blob[at: at + T * H], want)


def test_few_codes_in_a_plan_with_room_for_many_come_back(tsq):
    """Two bits of the eight that there is room for: 34 MB of codes where there is room for 134."""
    import torch
    T, H = 32768, 4096
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    x = torch.randn((T, H), device="cuda", generator=gen).half()
    plan = tsq.Plan(T, H, "f16", 8.0, (2, 8), 0.9, max_outliers=1024)
    blob = plan.compress(x.view(torch.int16))
    at, n = int(plan.layout.off_payload), int(plan.info(blob).payload_bytes)
    assert n == T * H // 4 and plan.layout.payload_capacity == T * H
    want = blob[at: at + n].clone()
    eblob = plan.entropy_encode(blob)
    blob[at: at + n] = 0xEE
    plan.entropy_decode(eblob, blob)
    assert torch.equal(blob[at: at + n], want)
