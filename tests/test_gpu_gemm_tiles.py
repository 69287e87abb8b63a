"""Products at the edges of the GEMM kernels' tiles and of the rule that picks them, against a float64 reference."""
import numpy as np
import pytest
import torch

from paper_2602_22732_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (1, 8, 64), (63, 65, 128), (65, 72, 192),      # one k-tile, fewer k-tiles than the ring of the 64x64 tiles, as many
    (128, 1028, 1024), (1025, 200, 320),           # columns past the last tile, columns that are no multiple of 8
    (2049, 3072, 192), (4100, 1000, 128),          # 128x128 tiles: paired and with a ragged edge
    (4096, 4096, 192), (4500, 3080, 256),          # few and many 256x256 tiles below 8192 rows
    (8200, 512, 192), (8192, 520, 256),            # the large class on 128x128 and on 256x256 tiles
    (2017, 1000, 64), (1030, 1500, 128),           # tiles that load for themselves, 64x64: one k-tile, fewer than LDS holds, ragged edges
    (500, 3001, 448), (4100, 1001, 192),           # as many and more; an odd number of columns
    (8191, 3080, 64), (4096, 4096, 128), (3000, 3001, 1024),  # 128x128: one k-tile, as many as LDS holds, more; ragged edges, odd columns
])
def test_linear_at_tile_edges(M, N, K):
    g = torch.Generator().manual_seed(M * 7 + N * 3 + K)
    A, W = torch.randn(M, K, generator=g).bfloat16(), (torch.randn(N, K, generator=g) / K**0.5).bfloat16()
    bias = torch.randn(N, generator=g)
    rows = torch.unique(torch.cat([torch.arange(min(M, 70)), torch.arange(max(0, M - 70), M), torch.randint(0, M, (60,), generator=g)]))
    ref = (A[rows].double() @ W.double().t()).numpy()
    a, w = A.cuda(), W.cuda()
    f32 = binding.op_linear(a, w, bias.cuda(), out_f32=True).cpu()[rows].double().numpy()
    half = binding.op_linear(a, w).cpu()[rows].double().numpy()
    np.testing.assert_allclose(f32, ref + bias.double().numpy(), atol=2e-5, rtol=1e-5)
    np.testing.assert_allclose(half, ref, atol=1e-6 + 2.0**-8 * np.abs(ref).max(), rtol=2.0**-7)


@pytest.mark.parametrize("M,N,K", [
    (1, 1, 4), (17, 33, 20), (16, 16, 512), (65, 130, 516),  # 16x16 tiles, K split over four wavefronts: empty and ragged shares
    (1024, 1024, 64), (2100, 520, 68),                       # 64x64 tiles
])
def test_f32_linear_at_tile_edges(M, N, K):
    g = torch.Generator().manual_seed(M + N + K)
    A, W, bias = torch.randn(M, K, generator=g), torch.randn(N, K, generator=g) / K**0.5, torch.randn(N, generator=g)
    out = binding.op_linear(A.cuda(), W.cuda(), bias.cuda(), out_f32=True).cpu().double()
    np.testing.assert_allclose(out.numpy(), (A.double() @ W.double().t() + bias.double()).numpy(), atol=1e-5, rtol=1e-6)


@pytest.mark.parametrize("N,K", [(1024, 4), (1040, 68), (1024, 132), (1032, 516), (1024, 1024)])
def test_f32_rows_do_not_depend_on_the_row_count(N, K):
    """Enough rows for the 64x64 tiles and few of them alone: the same bits."""
    g = torch.Generator().manual_seed(N + K)
    a, w = torch.randn(1100, K, generator=g).cuda(), torch.randn(N, K, generator=g).cuda()
    many = binding.op_linear(a, w, out_f32=True)
    for first, rows in ((0, 1), (37, 64), (1000, 100)):
        assert torch.equal(binding.op_linear(a[first:first + rows].contiguous(), w, out_f32=True), many[first:first + rows])


@pytest.mark.parametrize("d,H", [(128, 4), (384, 3), (1088, 17)])  # the last: gains past what the norm keeps in LDS
def test_f32_requests_do_not_depend_on_their_batch(d, H):
    """Products, norms and attention of one request alone and inside a batch whose products run on the larger tiles."""
    w = synth.Workload("batch", "f32", 40, 33, d, 3, 1, H, 2 * d, 3, [512, 264, 1024], [64, 64, 64], len_min=5)
    dec = binding.decoder_for(w, synth.make_weights(w))
    lens = synth.make_lengths(w, seed=1)
    ctx, cl = torch.from_numpy(synth.make_context(w, lens)).cuda(), torch.from_numpy(lens).int().cuda()
    sid, lp = dec.decode_batch(ctx, cl, w.beam)
    for b in (0, 39):
        one = dec.decode_batch(ctx[b:b + 1].contiguous(), cl[b:b + 1].contiguous(), w.beam)
        assert torch.equal(one[0][0], sid[b]) and torch.equal(one[1][0], lp[b])
    dec.close()


@pytest.mark.parametrize("N,K", [
    (512, 64), (520, 448), (512, 512), (1032, 576),  # one k-tile; one less than, as many as and one more than the deepest ring; ragged columns
    (3072, 1088), (264, 4096),
])
def test_bf16_rows_do_not_depend_on_the_row_count(N, K):
    """Below 8192 rows every kernel that runs a product adds in one order: rows alone, on small tiles, and among many, on larger ones, give the same bits."""
    g = torch.Generator().manual_seed(N + K)
    a, w = torch.randn(8000, K, generator=g).bfloat16().cuda(), (torch.randn(N, K, generator=g) / K**0.5).bfloat16().cuda()
    many, many32 = binding.op_linear(a, w), binding.op_linear(a, w, out_f32=True)
    for first, rows in ((0, 1), (37, 33), (100, 97), (1000, 300), (2000, 700), (3001, 1500), (4000, 4000)):
        some = a[first:first + rows].contiguous()
        assert torch.equal(binding.op_linear(some, w), many[first:first + rows])
        assert torch.equal(binding.op_linear(some, w, out_f32=True), many32[first:first + rows])
    np.testing.assert_allclose(many32[:64].double().cpu().numpy(), (a[:64].double() @ w.double().t()).cpu().numpy(), atol=2e-5, rtol=1e-5)


@pytest.mark.parametrize("d,H,F", [(256, 8, 1024), (512, 4, 2048), (1024, 16, 2048)])
@pytest.mark.parametrize("B,n", [(3, 33), (47, 33), (97, 31), (239, 33)])
def test_requests_do_not_depend_on_their_batch(d, H, F, B, n):
    """The products that add a residual or a table row: one request's rows on the smallest tiles, those of a batch (99 to 7887, ragged) on all the others."""
    w = synth.Workload("tiles", "bf16", B, 40, d, 3, 1, H, F, 3, [512, 300, 264], [n, n, n])
    dec = binding.decoder_for(w, synth.make_weights(w))
    ctx = torch.randn(B, 40, d, generator=torch.Generator(device="cuda").manual_seed(B + d), device="cuda").bfloat16()
    sid, lp = dec.decode_batch(ctx, None, w.beam)
    for b in (0, B // 2, B - 1):
        one = dec.decode_batch(ctx[b:b + 1].contiguous(), None, w.beam)
        assert torch.equal(one[0][0], sid[b]) and torch.equal(one[1][0], lp[b])
    assert torch.isfinite(lp).all()
    dec.close()
