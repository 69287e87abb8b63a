"""Levels whose token-only part runs on their distinct (request, previous token) rows.

FP8 products compute the same at every row count, so the same requests decoded in a batch below the size from which levels share rows
(8192) must come out bit for bit; bf16 decodes are held to the oracle and, bit for bit, to decodes that compute every row."""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_common import gpu_decode, judge_decode, judge_value, value_rounding_model
from paper_2602_22732_amd import binding, synth
from rounding_model import RoundedModel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,beam,V,Ve,vanilla", [
    (130, [64, 64, 64, 64], [64, 5, 70, 3000], 0, False),    # 5 and at most 70 tokens for 64 beams
    (129, [65, 67, 66, 65], [4096] * 4, 0, False),           # odd beams, few shared tokens
    (140, [64, 64, 30], [80, 300, 256], 64, False),          # the value step shares too (n = 30: below the size)
    (70, [120, 110, 127], [600, 90, 256], 64, False),        # the value step alone
    (70, [300, 300, 520], [600, 90, 256], 64, False),        # several blocks of beams, shared in both batches, packed differently
    (130, [64, 64, 64], [128, 16, 256], 0, True),            # vanilla input states
])
def test_fp8_decode_equals_the_same_requests_in_a_small_batch(B, beam, V, Ve, vanilla):
    w = synth.Workload("distinct", "bf16", B, 70, 512, 3, 0 if vanilla else 1, 8, 1024, len(V), V, beam, zipf_bias=True, fp8=True, Ve=Ve, vanilla=vanilla)
    dec = binding.decoder_for(w, synth.make_weights(w))
    g = torch.Generator(device="cuda").manual_seed(B)
    ctx = torch.randn(B, w.S, w.d, generator=g, device="cuda").bfloat16()
    lens = torch.randint(1, w.S + 1, (B,), generator=g, device="cuda").int()
    some = dec.decode_batch(ctx, lens, w.beam, value=bool(Ve))
    m = 64  # (at least as many rows as the FP8 matrix-core kernel takes, at level 1)
    few = dec.decode_batch(ctx[:m].contiguous(), lens[:m].contiguous(), w.beam, value=bool(Ve))
    torch.cuda.synchronize()
    for a, b in zip(some, few):
        assert torch.equal(a[:m], b)
    dec.close()


def profiled(dec, *args, **kw):
    binding.profile_read(reset=True)
    binding.profile_enable(True)
    out = dec.decode_batch(*args, **kw)
    prof = binding.profile_read(reset=True)
    binding.profile_enable(False)
    return out, "distinct_rows" in prof


@pytest.mark.parametrize("d,V,Ve,vanilla", [(256, [64, 6, 256, 300], 0, False), (512, [300, 300, 300], 0, False), (256, [64, 40, 264], 256, False),
                                            (256, [64, 7, 256], 0, True)])
def test_bf16_decode_equals_one_that_computes_every_row(d, V, Ve, vanilla):
    """(Sharing needs classifiers of 256 columns.)  Levels share rows only where the FFN is wide enough to lend its hidden rows; a narrower one is the same function as a wide one whose further hidden
    units are zero, so the two models give the same bits, one with and one without shared rows."""
    T, F = len(V), d
    w = synth.Workload("distinct", "bf16", 131, 40, d, 3, 0 if vanilla else 1, d // 64, F, T, V, [64] * T, len_min=3, zipf_bias=True, Ve=Ve, vanilla=vanilla)
    W = synth.make_weights(w)
    lens = synth.make_lengths(w, seed=3)
    ctx, cl = torch.from_numpy(synth.make_context(w, lens)).to("cuda", torch.bfloat16), torch.from_numpy(lens).int().cuda()
    dec = binding.decoder_for(w, W)
    every, found = profiled(dec, ctx, cl, w.beam, value=bool(Ve))
    assert not found
    dec.close()
    wide = dataclasses.replace(w, F=2 * F)
    pad = dict(W, layers=[dict(lw, w1=np.pad(lw["w1"], ((0, F), (0, 0))), w2=np.pad(lw["w2"], ((0, 0), (0, F)))) for lw in W["layers"]])
    dec = binding.decoder_for(wide, pad)
    shared, found = profiled(dec, ctx, cl, w.beam, value=bool(Ve))
    assert found
    torch.cuda.synchronize()
    for a, b in zip(shared, every):
        assert torch.equal(a, b)
    dec.close()


@pytest.mark.parametrize("V,Ve,vanilla", [([64, 6, 200, 96], 0, False), ([64, 6, 256, 300], 0, False), ([512, 512, 512], 0, False), ([64, 40, 64], 32, False),
                                          ([64, 40, 264], 256, False), ([64, 7, 256], 0, True)])
def test_bf16_decode_matches_oracle(V, Ve, vanilla):
    T = len(V)
    w = synth.Workload("distinct", "bf16", 131, 20, 256, 2, 0 if vanilla else 1, 4, 512, T, V, [64] * T, len_min=3, zipf_bias=True, Ve=Ve, vanilla=vanilla)
    W = synth.make_weights(w)
    lens = synth.make_lengths(w, seed=3)
    X = synth.make_context(w, lens)
    res = gpu_decode(w, W, X, lens, value=bool(Ve))
    print(judge_decode(w, W, X, lens, res[0], res[1], res[2], [0, 65, 130], model=RoundedModel(w, W)))
    if Ve:
        print(judge_value(w, W, X, lens, res[0], res[1], res[3], [130], model=value_rounding_model(w, W)))
    assert np.isfinite(res[1]).all()


def test_captured_replays_match_eager_calls():
    """The number of distinct rows is read on the device, so a captured decode follows new contexts."""
    w = synth.Workload("distinct", "bf16", 131, 20, 256, 2, 1, 4, 512, 3, [512, 512, 512], [64] * 3, len_min=3, zipf_bias=True)
    dec = binding.decoder_for(w, synth.make_weights(w))
    g = torch.Generator(device="cuda").manual_seed(5)
    ctx = torch.randn(w.B, w.S, w.d, generator=g, device="cuda").bfloat16()
    ws = torch.empty(dec.workspace_bytes(w.B, w.S, w.beam), dtype=torch.uint8, device="cuda")
    sid = torch.empty(w.B, 64, 3, dtype=torch.int32, device="cuda")
    lp = torch.empty(w.B, 64, dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        dec.decode_batch(ctx, None, w.beam, workspace=ws, out_sid=sid, out_logprob=lp)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        dec.decode_batch(ctx, None, w.beam, workspace=ws, out_sid=sid, out_logprob=lp)
    for _ in range(3):
        ctx.copy_(torch.randn(w.B, w.S, w.d, generator=g, device="cuda"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = sid.clone(), lp.clone()
        want = dec.decode_batch(ctx, None, w.beam)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    dec.close()


def test_profiled_decode_counts_distinct_rows_without_waiting():
    """The timing counts the work of the rows that are there, and a profiled call only enqueues work like any other."""
    B, n, S, d, L, K, T = 130, 64, 70, 512, 4, 1, 4
    w = synth.Workload("distinct", "bf16", B, S, d, L, K, 8, 1024, T, [64, 5, 70, 300], [n] * T, zipf_bias=True, fp8=True)
    dec = binding.decoder_for(w, synth.make_weights(w))
    ctx = torch.randn(B, S, d, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda").bfloat16()
    tr = dec.enable_trace(B, w.beam)
    dec.decode_batch(ctx, None, w.beam)
    torch.cuda.synchronize()
    binding.profile_read(reset=True)
    binding.profile_enable(True)
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    for _ in range(200):  # some tenths of a second of work in front
        a @ a
    busy = torch.cuda.Event()
    busy.record()
    dec.decode_batch(ctx, None, w.beam)
    waited = busy.query()
    prof = binding.profile_read(reset=True)
    binding.profile_enable(False)
    assert not waited
    want = 0.0
    for t in range(T):
        rows = B * (n if t else 1)
        first = rows
        if t >= 2:  # a request's beams share their previous tokens
            first = sum(len(torch.unique(tr["tok"][t - 1][b])) for b in range(B))
        want += 4.0 * S * d * (first + (L - K - 1) * rows)
    assert abs(prof["cross_attn_flash_bf16"]["flops"] / want - 1) < 1e-9
    dec.close()
