"""Lazy layers of a few requests, whose context attention runs its tiles side by side: against the one-pass kernel, bit for bit.

A decode whose batch is large enough runs the one-pass kernel, so the same requests decoded alone and inside such a batch go through
both; a request's result does not depend on its batch."""
import pytest
import torch

from paper_2602_22732_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H,T,S,lens", [
    (512, 8, 3, 300, [1, 31, 32, 33, 255, 256, 257, 300]),   # one query tile: edges of tiles, stages and chunks
    (512, 8, 7, 64, [64, 1, 40]),                             # two query tiles, one stage
    (1024, 16, 4, 290, [290, 289, 3, 128]),                   # 64 queries
    (1024, 16, 5, 96, [96, 65]),                              # 80 queries: two launches
    (512, 8, 3, 100, list(range(1, 101)) + [100] * 28),       # as many requests as run side by side: several tiles to a workgroup
    (512, 8, 7, 300, [300 - 7 * i for i in range(40)] + [300] * 24),
    (1024, 16, 4, 290, [290 - 6 * i for i in range(48)]),
])
def test_few_requests_equal_the_same_requests_in_a_large_batch(d, H, T, S, lens):
    n, big = len(lens), 65536 // d + 1
    w = synth.Workload("split", "bf16", big, S, d, 2, 1, H, 256, T, [64] * T, [2] * T)
    dec = binding.decoder_for(w, synth.make_weights(w))
    g = torch.Generator(device="cuda").manual_seed(d + S)
    ctx = torch.randn(big, S, d, generator=g, device="cuda").bfloat16()
    length = torch.tensor(lens + [1] * (big - n), dtype=torch.int32, device="cuda")
    sid, lp = dec.decode_batch(ctx, length, w.beam)
    few_sid, few_lp = dec.decode_batch(ctx[:n].contiguous(), length[:n].contiguous(), w.beam)
    torch.cuda.synchronize()
    assert torch.equal(few_sid, sid[:n]) and torch.equal(few_lp, lp[:n])
    dec.close()


@pytest.mark.parametrize("d,H,most", [(512, 8, 128), (1024, 16, 48)])
def test_workspace_of_a_larger_batch_serves_a_smaller_one(d, H, most):
    """Across the batch size from which the lazy layers need no scratch of their own."""
    w = synth.Workload("split", "bf16", most + 2, 64, d, 2, 1, H, 256, 3, [64] * 3, [2] * 3)
    dec = binding.decoder_for(w, synth.make_weights(w))
    sizes = [dec.workspace_bytes(B, w.S, w.beam) for B in range(most - 2, most + 3)]
    assert sizes == sorted(sizes)
    ctx = torch.randn(most, w.S, d, generator=torch.Generator(device="cuda").manual_seed(d), device="cuda").bfloat16()
    sid, lp = dec.decode_batch(ctx, None, w.beam, workspace=torch.empty(sizes[3], dtype=torch.uint8, device="cuda"))
    want = dec.decode_batch(ctx, None, w.beam)
    torch.cuda.synchronize()
    assert torch.equal(sid, want[0]) and torch.equal(lp, want[1])
    dec.close()
