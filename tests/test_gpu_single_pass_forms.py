"""The two forms of the single-pass compress (one workgroup per token; persistent workgroups) at the shapes where they
can go wrong: both sides of the line between them, edges of the placement's blocks of 2048 tokens, the last run
of a row cut short, tokens with more outliers than a wave keeps in LDS, more tokens than one launch can have workgroups
for.  Whole blobs against the oracle."""
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


def kernel_of(tsq, T, H, dtype):
    return tsq.tsq_plan_kernel(tsq.Plan(T, H, dtype, 6.0, (2, 4, 8), 0.05, pipeline="fused").handle)


# rows that fill their waves and rows that do not, per kernel; only the persistent one keeps outliers in LDS
@pytest.mark.parametrize("T,H,dtype,kernel", [(40, 4096, "f16", "k_direct"), (40, 1032, "bf16", "k_direct"),
                                              (3200, 4096, "f16", "k_direct"), (1600, 8192, "bf16", "k_direct"),
                                              (5000, 4096, "f16", "k_fused"), (4300, 4088, "bf16", "k_fused"),
                                              (2800, 6000, "f16", "k_fused"), (2200, 8192, "bf16", "k_fused"),
                                              (1200, 8200, "f16", "k_fused"), (600, 32768, "bf16", "k_fused")])
def test_tokens_full_of_outliers(tsq, oracle, T, H, dtype, kernel):
    assert kernel_of(tsq, T, H, dtype) == kernel
    ref, _ = check_parity(tsq, oracle, rows(T, H, dtype, heavy=30), dtype, 6.0, (2, 4, 8), 0.05, "rel_rms", "fused",
                          label="heavy rows T=%d H=%d" % (T, H))
    assert np.diff(ref.row_ptr.astype(np.int64)).max() == H


# more tokens than the device holds workgroups for, so that tickets are drawn: every number of waves, both types,
# whole and ragged rows, both return rules, both modes
@pytest.mark.parametrize("T,H,dtype,mode,rule", [
    (4400, 4096, "bf16", "rel_rms", "as_printed"), (9001, 4088, "f16", "lsb", "last_passing"),
    (5600, 6144, "f16", "rel_rms", "as_printed"), (3001, 5000, "bf16", "lsb", "as_printed"),
    (2300, 8192, "f16", "rel_rms", "last_passing"), (4001, 6152, "bf16", "rel_rms", "as_printed"),
    (1100, 16384, "f16", "rel_rms", "last_passing"), (1501, 8200, "bf16", "lsb", "as_printed"),
    (700, 32768, "f16", "rel_rms", "as_printed"), (601, 16392, "bf16", "lsb", "last_passing")])
def test_the_persistent_form_at_every_number_of_waves(tsq, oracle, T, H, dtype, mode, rule):
    assert kernel_of(tsq, T, H, dtype) == "k_fused"
    ref, _ = check_parity(tsq, oracle, rows(T, H, dtype), dtype, 6.0, (2, 3, 4, 5, 6, 8), 0.2, mode, "fused",
                          label="T=%d H=%d" % (T, H), rule=rule)
    assert len(set(ref.bits.tolist())) > 1


@pytest.mark.parametrize("T", [2 ** 26 - 4096, 2 ** 26])
def test_as_many_tokens_as_a_launch_has_threads_for(tsq, oracle, T):
    """A launch's threads are counted in 32 bits, which ends one workgroup per token of one wave at 2^26 - 1 tokens: the
    last thousands below that, and the first count beyond it.  The tokens are copies of a block of 4096, so every section
    is the block's over and over, the offsets moved on by the block's totals; compared on the card."""
    import torch
    H, B = 8, 4096
    x = rows(B, H, "f16")
    ref = oracle.compress(x, oracle.F16, 6.0, (2, 4, 8), 0.05, 1, nthreads=8)
    assert ref.nnz > 0 and len(set(ref.bits.tolist())) > 1
    copies = T // B
    plan = tsq.Plan(T, H, "f16", 6.0, (2, 4, 8), 0.05, pipeline="fused", max_outliers=copies * ref.nnz)
    xd = torch.from_numpy(x.view(np.int16)).cuda().repeat(copies, 1)
    blob, ws = plan.new_blob(), plan.new_workspace()
    torch.cuda.synchronize()
    print("compress", T, "tokens", flush=True)
    plan.compress(xd, blob, ws)
    info = plan.info(blob)
    assert info.status == 0 and info.nnz == copies * ref.nnz and info.payload_bytes == copies * ref.payload_bytes
    L = plan.layout

    def same(at, want, dtype):
        w = torch.from_numpy(want.view(np.uint8).copy()).cuda().view(dtype)
        got = blob[int(at):int(at) + copies * w.numel() * w.element_size()].view(dtype).view(copies, w.numel())
        return bool((got == w).all())

    assert same(L.off_bits, ref.bits, torch.uint8) and same(L.off_scale, ref.scale, torch.int32)
    assert same(L.off_payload, ref.payload, torch.uint8)
    assert same(L.off_out_col, ref.out_col, torch.int16) and same(L.off_out_val, ref.out_val, torch.int16)
    for at, want, total in ((L.off_pay_off, ref.pay_off, ref.payload_bytes), (L.off_row_ptr, ref.row_ptr, ref.nnz)):
        got = blob[int(at):int(at) + 8 * T].view(torch.int64).view(copies, B)
        w = torch.from_numpy(want[:B].astype(np.int64)).cuda()
        assert bool((got == w + total * torch.arange(copies, device="cuda").view(-1, 1)).all())
        assert int(blob[int(at) + 8 * T:int(at) + 8 * (T + 1)].view(torch.int64)) == copies * total
