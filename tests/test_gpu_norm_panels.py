"""Products that form their own rows - norms, gated rows, the trunk's self-attention - (at most 1024 columns, few tiles): the same bits as the kernels of their own that many
rows take."""
import pytest
import torch

from paper_2602_22732_amd import binding, synth

pytestmark = pytest.mark.gpu


# Norms: the first FFN product of the batch, which takes 2048 columns, runs behind the norm kernel, the others' rows are formed by the product on either side.
# d: one k-tile, less than the 256 columns that two rows share a wavefront for, as many, more, as many as 512, more (where 16 rows are the most), as many as 1024.
# n: the rows of one wavefront step, one more, two steps, one more, a second tile of 32 rows
@pytest.mark.parametrize("d,H", [(64, 1), (128, 8), (192, 3), (256, 8), (320, 5), (512, 8), (576, 9), (1024, 16)])
@pytest.mark.parametrize("n", [8, 9, 16, 17, 33])
def test_requests_do_not_depend_on_their_batch(d, H, n):
    B = 1200 // n
    w = synth.Workload("panels", "bf16", B, 40, d, 3, 1, H, 2048, 3, [512, 300, 264], [n, n, n])
    dec = binding.decoder_for(w, synth.make_weights(w))
    ctx = torch.randn(B, 40, d, generator=torch.Generator(device="cuda").manual_seed(n + d), device="cuda").bfloat16()
    sid, lp = dec.decode_batch(ctx, None, w.beam)
    for b in (0, B - 1):
        one = dec.decode_batch(ctx[b:b + 1].contiguous(), None, w.beam)
        assert torch.equal(one[0][0], sid[b]) and torch.equal(one[1][0], lp[b])
    assert torch.isfinite(lp).all()
    dec.close()


def launches(dec, ctx, beam):
    """The decode and its launches of the trunk's self-attention and of Fuse's gate."""
    binding.profile_enable(True)
    try:
        binding.profile_read()
        out = dec.decode_batch(ctx, None, beam)
        torch.cuda.synchronize()
        count = {k: v["launches"] for k, v in binding.profile_read().items()}
    finally:
        binding.profile_enable(False)
    return out, count.get("trunk_self_attn", 0), count.get("fuse_gate", 0)


# Gates and the trunk's self-attention: in the batch both run as kernels of their own - the gates of all levels but the first -, in the few requests of `few` both are formed by the product.
# Head widths 16, 32 and 64, three and four positions; d: two rows to a wavefront with 8 (d = 64) to 32 (256) pieces of a row, one row of up to 64 pieces, of up to 128.
# few: trunk and gated rows on all tile shapes: up to 8 and up to 16 rows, 32x32, 32x64 and, gated, 64x64 tiles.
@pytest.mark.parametrize("dh", [16, 32, 64])
@pytest.mark.parametrize("d,T,B,n,few", [(64, 3, 2800, 3, (1, 8, 100, 400)), (128, 3, 2800, 3, (1, 8, 100, 400)), (192, 3, 2800, 3, (1, 8, 100, 400)), (256, 3, 700, 9, (1, 8, 100, 400)),
                                         (256, 4, 520, 13, (1, 4, 8, 100)), (320, 4, 200, 9, (1, 2, 4)), (512, 3, 140, 8, (1, 2, 5)), (576, 3, 40, 8, (1, 2)), (1024, 4, 40, 8, (1, 2))])
def test_gates_and_trunk_attention_as_their_own_kernels(d, T, B, n, few, dh):
    # (192 columns of the FFN and 200 tokens: no product of a class that rounds differently)
    w = synth.Workload("rows", "bf16", B, 8, d, 3, 1, d // dh, 192, T, [200] * T, [n] * T)
    dec = binding.decoder_for(w, synth.make_weights(w))
    ctx = torch.randn(B, 8, d, generator=torch.Generator(device="cuda").manual_seed(d + dh), device="cuda").bfloat16()
    (sid, lp), trunk, gates = launches(dec, ctx, w.beam)
    assert torch.isfinite(lp).all() and trunk == w.K and gates >= T - 1
    for b in few:
        (few_sid, few_lp), trunk, gates = launches(dec, ctx[B - b:].contiguous(), w.beam)
        assert (trunk, gates) == (0, 0)
        assert torch.equal(few_sid, sid[B - b:]) and torch.equal(few_lp, lp[B - b:])
    dec.close()
