"""Short rows, eight tokens a workgroup (rows of two waves: two): token counts around the first that takes that form, around
whole groups and around a block of 2048 groups; rows that fill their wave, that end inside a run, and of a single piece;
tokens full of outliers; a table of tensors; a workspace of another shape.  Whole blobs against the oracle."""
import numpy as np
import pytest

from test_gpu_parity import check_parity, tsq  # noqa: F401
from test_gpu_single_pass_forms import kernel_of, rows

pytestmark = pytest.mark.gpu


def per_workgroup(tsq, T, H, dtype):
    return tsq.tsq_plan_direct_launch(tsq.Plan(T, H, dtype, 6.0, (2, 4, 8), 0.05, pipeline="fused").handle)[0]


@pytest.mark.parametrize("T,H,dtype", [(1023, 2048, "f16"), (1024, 2048, "bf16"), (1025, 2048, "f16"), (1031, 2040, "bf16"),
                                       (1032, 1032, "f16"), (2049, 768, "bf16"), (4095, 520, "f16"), (16383, 264, "bf16"),
                                       (16384, 256, "f16"), (16385, 256, "bf16"), (16393, 40, "f16"), (32771, 8, "bf16")])
def test_token_counts_around_groups_and_blocks(tsq, oracle, T, H, dtype):
    assert kernel_of(tsq, T, H, dtype) == "k_direct"
    assert per_workgroup(tsq, T, H, dtype) == (1 if T < 1024 else 8)
    check_parity(tsq, oracle, rows(T, H, dtype), dtype, 6.0, (2, 3, 4, 6, 8), 0.1, "rel_rms", "fused", label="T=%d H=%d" % (T, H))


@pytest.mark.parametrize("T,H,dtype,mode,rule", [(1500, 2048, "f16", "lsb", "as_printed"), (2001, 1000, "bf16", "rel_rms", "as_printed"),
                                                 (1999, 776, "f16", "rel_rms", "last_passing"), (3003, 2048, "bf16", "lsb", "last_passing")])
def test_groups_with_tokens_full_of_outliers(tsq, oracle, T, H, dtype, mode, rule):
    ref, _ = check_parity(tsq, oracle, rows(T, H, dtype, heavy=40), dtype, 6.0, (2, 3, 4, 5, 6, 8), 0.2, mode, "fused",
                          label="heavy T=%d H=%d" % (T, H), rule=rule)
    assert np.diff(ref.row_ptr.astype(np.int64)).max() == H


def test_groups_over_a_table_of_tensors(tsq, oracle):
    import torch
    T, H, n = 1365, 1024, 13                                  # tensors end inside groups
    x = rows(T, H, "f16")
    ref = oracle.compress(x, oracle.F16, 6.0, (2, 4, 8), 0.1, 1, nthreads=8)
    plan = tsq.Plan(T, H, "f16", 6.0, (2, 4, 8), 0.1, max_outliers=ref.nnz)
    parts = [torch.from_numpy(x[i * (T // n):(i + 1) * (T // n)].view(np.int16).copy()).cuda() for i in range(n)]
    blob, ws = plan.new_blob(), plan.new_workspace()
    plan.compress_batch(parts, blob, ws)
    assert plan.info(blob).status == 0
    sec = plan.sections(blob)
    for k in ("bits", "pay_off", "row_ptr", "payload", "out_col", "out_val"):
        assert np.array_equal(sec[k], getattr(ref, k)), k


@pytest.mark.parametrize("T,H", [(1087, 264), (1088, 264), (1089, 264), (1151, 2048), (1024, 8)])
def test_restore_writes_every_row_of_such_a_call_once(tsq, oracle, T, H):
    # the order in which restore takes the tokens follows the groups: counts around the multiples of 64 where it changes
    import torch
    x = rows(T, H, "bf16")
    ref = oracle.compress(x, oracle.BF16, 6.0, (2, 4, 8), 0.1, 1, nthreads=8)
    plan = tsq.Plan(T, H, "bf16", 6.0, (2, 4, 8), 0.1, max_outliers=ref.nnz)
    blob, ws = plan.new_blob(), plan.new_workspace()
    plan.compress(torch.from_numpy(x.view(np.int16).copy()).cuda(), blob, ws)
    want = oracle.decompress(ref, nthreads=8)
    assert np.array_equal(plan.decompress(blob).cpu().numpy().view(np.uint16), want)
    if T % 17 == 0:
        outs = [torch.zeros((T // 17, H), dtype=torch.int16, device="cuda") for _ in range(17)]
        plan.decompress_batch(blob, outs)
        assert np.array_equal(torch.cat(outs).cpu().numpy().view(np.uint16), want)


@pytest.mark.parametrize("T,H,dtype,mode,rule,heavy", [
    (1023, 4096, "f16", "rel_rms", "last_passing", 0), (1024, 4096, "bf16", "rel_rms", "as_printed", 0),
    (1025, 2056, "f16", "lsb", "as_printed", 0), (1280, 4088, "bf16", "rel_rms", "last_passing", 40),
    (1281, 4088, "bf16", "rel_rms", "last_passing", 40), (1281, 2056, "f16", "lsb", "as_printed", 0), (1535, 2856, "bf16", "lsb", "last_passing", 40),
    (2049, 4088, "f16", "rel_rms", "as_printed", 40), (4095, 2080, "bf16", "rel_rms", "last_passing", 0),
    (4096, 4096, "f16", "lsb", "as_printed", 0)])
def test_rows_of_two_waves_two_tokens_a_workgroup(tsq, oracle, T, H, dtype, mode, rule, heavy):
    # both tokens of a workgroup go through the widths together: many widths, tokens that leave at different ones; whole
    # blocks of 2048 groups; a last group of one token
    assert kernel_of(tsq, T, H, dtype) == "k_direct"
    assert per_workgroup(tsq, T, H, dtype) == (2 if T >= (1024 if H == 4096 else 1281) else 1)
    x = rows(T, H, dtype, heavy=heavy) if heavy else rows(T, H, dtype)
    check_parity(tsq, oracle, x, dtype, 6.0, (2, 3, 4, 5, 6, 8), 0.2, mode, "fused", label="T=%d H=%d" % (T, H), rule=rule)


@pytest.mark.parametrize("H,dtype", [(4096, "f16"), (2856, "bf16")])
def test_pairs_over_a_table_of_tensors(tsq, oracle, H, dtype):
    import torch
    T, n = 1365, 13                                           # tensors of 105 rows end inside pairs
    assert per_workgroup(tsq, T, H, dtype) == 2
    x = rows(T, H, dtype)
    ref = oracle.compress(x, oracle.F16 if dtype == "f16" else oracle.BF16, 6.0, (2, 4, 8), 0.1, 1, nthreads=8)
    plan = tsq.Plan(T, H, dtype, 6.0, (2, 4, 8), 0.1, max_outliers=ref.nnz)
    parts = [torch.from_numpy(x[i * (T // n):(i + 1) * (T // n)].view(np.int16).copy()).cuda() for i in range(n)]
    blob, ws = plan.new_blob(), plan.new_workspace()
    plan.compress_batch(parts, blob, ws)
    assert plan.info(blob).status == 0
    sec = plan.sections(blob)
    for k in ("bits", "pay_off", "row_ptr", "payload", "out_col", "out_val"):
        assert np.array_equal(sec[k], getattr(ref, k)), k
    outs = [torch.zeros((T // n, H), dtype=torch.int16, device="cuda") for _ in range(n)]
    plan.decompress_batch(blob, outs)
    assert np.array_equal(torch.cat(outs).cpu().numpy().view(np.uint16), oracle.decompress(ref, nthreads=8))


@pytest.mark.parametrize("T,fewer,H,tokens", [(1500, 1100, 2048, 8), (1031, 1024, 776, 8), (2100, 1101, 4096, 2), (1501, 1300, 2856, 2)])
def test_groups_leave_a_workspace_of_another_shape_alone(tsq, oracle, T, fewer, H, tokens):
    """A workspace of all-ones bytes and one of a smaller plan: a header with TSQ_ERR_FORMAT and nothing else, the workspace
    keeps every byte and still serves the plan it was reset for."""
    import torch
    assert per_workgroup(tsq, T, H, "f16") == per_workgroup(tsq, fewer, H, "f16") == tokens
    x = rows(T, H, "f16")
    xd = torch.from_numpy(x.view(np.int16)).cuda()
    plan, small = (tsq.Plan(n, H, "f16", 6.0, (2, 4, 8), 0.1, pipeline="fused") for n in (T, fewer))
    blob = plan.new_blob().zero_()
    never = torch.full((int(plan.layout.workspace_bytes),), 0xFF, dtype=torch.uint8, device="cuda")
    ws = small.new_workspace()
    torch.cuda.synchronize()
    before = ws.clone()
    for name, w, want in (("all-ones bytes", never, never.clone()), ("a smaller plan's workspace", ws, before)):
        print("compress on", name, flush=True)
        plan.compress(xd, blob, w)
        info = plan.info(blob, check=False)
        assert info.return_status == tsq.TSQ_ERR_FORMAT and info.status == tsq.TSQ_ERR_FORMAT
        assert torch.equal(w, want)
        assert not bool(blob[int(plan.layout.off_bits):].any())
    out = torch.full((T, H), 0x1234, dtype=torch.int16, device="cuda")
    plan.decompress(blob, out)                                # refused: the output stays as it was
    torch.cuda.synchronize()
    assert bool((out == 0x1234).all())
    ref = oracle.compress(x[:fewer], oracle.F16, 6.0, (2, 4, 8), 0.1, 1, nthreads=8)
    b2 = small.compress(xd[:fewer].contiguous(), None, ws)
    assert small.info(b2).status == 0
    sec = small.sections(b2)
    for k in ("bits", "pay_off", "row_ptr", "payload", "out_col", "out_val"):
        assert np.array_equal(sec[k], getattr(ref, k)), k


@pytest.mark.parametrize("T,tokens", [(2 ** 26 - 8, 8), (2 ** 26 - 1, 1)])
def test_the_most_tokens_that_groups_and_single_tokens_take(tsq, oracle, T, tokens):
    """A launch's threads are counted in 32 bits: the last token count whose groups fit that, and the last that a workgroup
    per token does.  The tokens are copies of a block of 4096 and the front of one; compared on the card."""
    import torch
    H, B = 8, 4096
    x = rows(B, H, "f16")
    copies, rest = divmod(T, B)
    ref = oracle.compress(x, oracle.F16, 6.0, (2, 4, 8), 0.05, 1, nthreads=8)
    end = oracle.compress(x[:rest], oracle.F16, 6.0, (2, 4, 8), 0.05, 1, nthreads=8)
    assert end.nnz > 0 and len(set(end.bits.tolist())) > 1
    nnz = copies * ref.nnz + end.nnz
    plan = tsq.Plan(T, H, "f16", 6.0, (2, 4, 8), 0.05, pipeline="fused", max_outliers=nnz)
    assert tsq.tsq_plan_direct_launch(plan.handle)[0] == tokens
    xd = torch.from_numpy(x.view(np.int16)).cuda().repeat(copies + 1, 1)[:T]
    blob, ws = plan.new_blob(), plan.new_workspace()
    torch.cuda.synchronize()
    print("compress", T, "tokens", flush=True)
    plan.compress(xd, blob, ws)
    info = plan.info(blob)
    assert info.status == 0 and info.nnz == nnz and info.payload_bytes == copies * ref.payload_bytes + end.payload_bytes
    L = plan.layout

    for at, name in ((L.off_bits, "bits"), (L.off_scale, "scale"), (L.off_payload, "payload"), (L.off_out_col, "out_col"),
                     (L.off_out_val, "out_val")):
        w, e = (torch.from_numpy(getattr(r, name).view(np.uint8).copy()).cuda() for r in (ref, end))
        at, n = int(at), w.numel()
        assert bool((blob[at:at + copies * n].view(copies, n) == w).all()), name
        assert torch.equal(blob[at + copies * n:at + copies * n + e.numel()], e), name
    for at, name, total in ((L.off_pay_off, "pay_off", ref.payload_bytes), (L.off_row_ptr, "row_ptr", ref.nnz)):
        got = blob[int(at):int(at) + 8 * (T + 1)].view(torch.int64)
        w, e = (torch.from_numpy(getattr(r, name).astype(np.int64)).cuda() for r in (ref, end))
        assert bool((got[:copies * B].view(copies, B) == w[:B] + total * torch.arange(copies, device="cuda").view(-1, 1)).all()), name
        assert torch.equal(got[copies * B:], e + copies * total), name
