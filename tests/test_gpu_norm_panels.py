"""Products that form their own rows - norms, gated rows, the trunk's self-attention - (at most 1024 columns, few tiles): the same bits as the kernels of their own that many
rows take."""
import pytest
import torch

from paper_2602_22732_amd import binding, synth

pytestmark = pytest.mark.gpu


# d: one k-tile, less than the 256 columns that two rows share a wavefront for, as many, more, as many as 512, more (where 16 rows are the most), as many as 1024.
# n: the rows of one wavefront step, one more, two steps, one more, a second tile of 32 rows
@pytest.mark.parametrize("d,H", [(64, 1), (128, 8), (192, 3), (256, 8), (320, 5), (512, 8), (576, 9), (1024, 16)])
@pytest.mark.parametrize("n", [8, 9, 16, 17, 33])
def test_requests_do_not_depend_on_their_batch(d, H, n):
    B = 1200 // n  # (enough rows that the first FFN product, 2048 columns, runs behind the norm kernel)
    w = synth.Workload("panels", "bf16", B, 40, d, 3, 1, H, 2048, 3, [512, 300, 264], [n, n, n])
    dec = binding.decoder_for(w, synth.make_weights(w))
    ctx = torch.randn(B, 40, d, generator=torch.Generator(device="cuda").manual_seed(n + d), device="cuda").bfloat16()
    sid, lp = dec.decode_batch(ctx, None, w.beam)
    for b in (0, B - 1):
        one = dec.decode_batch(ctx[b:b + 1].contiguous(), None, w.beam)
        assert torch.equal(one[0][0], sid[b]) and torch.equal(one[1][0], lp[b])
    assert torch.isfinite(lp).all()
    dec.close()
