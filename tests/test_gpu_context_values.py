"""Context keys and values: products over all layers at once or layer by layer, on the persistent kernel or on small tiles, at context lengths
that are and are not multiples of 64.  A request's result does not depend on its batch, so a few requests alone (small tiles, all lazy layers
together) must equal, to the bit, the same requests in a batch whose products run on the persistent kernel, one lazy layer at a time."""
import pytest
import torch

from paper_2602_22732_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,L,K", [(8, 4, 2), (4, 3, 1)])  # head width 32: lazy layers with keys and values of their own; 64: absorbed
@pytest.mark.parametrize("B,S,low", [(300, 100, 1), (100, 389, 65), (700, 5, 1), (300, 128, 3), (600, 64, 64)])
def test_requests_alone_equal_the_same_requests_in_a_large_batch(H, L, K, B, S, low):
    w = synth.Workload("values", "bf16", B, S, 256, L, K, H, 512, 2, [64, 300], [4, 6])
    dec = binding.decoder_for(w, synth.make_weights(w))
    g = torch.Generator(device="cuda").manual_seed(B + S)
    ctx = torch.randn(B, S, 256, generator=g, device="cuda").bfloat16()
    lens = torch.randint(low, S + 1, (B,), generator=g, device="cuda").int()
    lens[0], lens[-1], lens[1] = S, S, low
    sid, lp = dec.decode_batch(ctx, lens, w.beam)
    for part in (slice(0, 5), slice(B - 3, B), slice(B // 2, B // 2 + 1)):
        few = dec.decode_batch(ctx[part].contiguous(), lens[part].contiguous(), w.beam)
        torch.cuda.synchronize()
        assert torch.equal(few[0], sid[part]) and torch.equal(few[1], lp[part])
    assert torch.isfinite(lp).all()
    dec.close()


def test_workspace_of_a_longer_or_larger_batch_serves_a_shorter_or_smaller_one():
    """Across the number of context rows up to which the lazy layers' keys and values are projected together."""
    w = synth.Workload("values", "bf16", 600, 130, 256, 7, 6, 8, 512, 2, [64, 300], [4, 6])
    dec = binding.decoder_for(w, synth.make_weights(w))
    for S in (1, 63, 64, 65, 100, 128):
        sizes = [dec.workspace_bytes(B, S, w.beam) for B in (1, 100, 255, 256, 257, 511, 512, 513, 600)]
        assert sizes == sorted(sizes)
    for B in (1, 255, 256, 257, 300, 512, 600):
        sizes = [dec.workspace_bytes(B, S, w.beam) for S in range(1, 130, 3)]
        assert sizes == sorted(sizes)
    dec.close()
