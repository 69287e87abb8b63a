"""Selections with scores that are no numbers: every request still gets k distinct candidates with tokens and parents in range.  With several
rows per request a row without numbers ranks below all numbers; a request of one row ranks as a selection without a bound does (the
order of the score keys, in which a NaN lies above or below all numbers by its sign)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import judge_selection
from paper_2602_22732_amd import binding, synth

pytestmark = pytest.mark.gpu


def unbounded(logits, cum, k):
    """The selection as the workgroup kernel makes it, which knows no bound: float32 logits that are not 16-byte aligned.  (Requests of one row: in one launch that adds a row up in
    that kernel's order.)"""
    buf = torch.empty(logits.size + 1, device="cuda")[1:]
    z = buf.view(logits.shape).copy_(torch.from_numpy(logits.astype(np.float32)))
    assert z.data_ptr() % 16
    return (t.cpu().numpy() for t in binding.op_select(z, torch.from_numpy(cum).cuda(), k))


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("kind", ["nan", "all_nan", "inf", "all_neg_inf", "cum_neg_inf", "cum_nan", "cum_inf"])
@pytest.mark.parametrize("where", ["first", "last", "every"])
@pytest.mark.parametrize("B,n,V,k", [(2, 1, 1024, 1024), (3, 1, 264, 7), (2, 3, 8192, 600), (2, 130, 264, 264)])
def test_select_of_scores_that_are_no_numbers(B, n, V, k, where, kind, half):
    rng = np.random.default_rng([B, n, V, k, half])
    logits = rng.standard_normal((B, n, V)).astype(np.float16 if half else np.float32)
    cum = (-2.0 * rng.random((B, n))).astype(np.float32)
    rows = {"first": [0], "last": [n - 1], "every": range(n)}[where]
    for i in rows:  # (the last request keeps numbers, where there is more than one)
        z, c = logits[:B - 1, i], cum[:B - 1, i]
        if kind == "nan":
            z[:, 5] = np.nan
        elif kind == "all_nan":
            z[:] = np.nan
        elif kind == "inf":
            z[:, V - 3] = np.inf
        elif kind == "all_neg_inf":
            z[:] = -np.inf
        else:
            c[:] = {"cum_neg_inf": -np.inf, "cum_nan": np.nan, "cum_inf": np.inf}[kind]
    print(kind, where, "half", half, "B n V k", B, n, V, k, flush=True)
    parent, tok, score = (t.cpu().numpy() for t in binding.op_select(torch.from_numpy(logits).cuda(), torch.from_numpy(cum).cuda(), k))
    u_parent, u_tok, u_score = unbounded(logits, cum, k)
    assert (parent >= 0).all() and (parent < n).all() and (tok >= 0).all() and (tok < V).all()
    for b in range(B):
        flat = parent[b].astype(np.int64) * V + tok[b]
        assert len(np.unique(flat)) == k
        with np.errstate(invalid="ignore"):
            want = cum[b].astype(np.float64)[:, None] + np.stack([oracle.prim_log_softmax(z) if np.abs(z).max() < np.inf else np.full(V, np.nan)
                                                                  for z in logits[b].astype(np.float32)])
        want = want.ravel()
        # +inf, then numbers, -inf and what is no number; ties in the order of the candidates
        up, numbers, down, none = (np.flatnonzero(w) for w in (want == np.inf, np.isfinite(want), want == -np.inf, np.isnan(want)))
        assert len(none) == 0 or n == 1 or len(up) + len(numbers) + len(down) >= k or where == "every"
        if n == 1 and len(none):
            u_flat = u_parent[b].astype(np.int64) * V + u_tok[b]
            assert np.array_equal(flat, u_flat) and np.array_equal(score[b], u_score[b], equal_nan=True)
            continue
        take = [len(up[:k])]
        for part in (numbers, down, none):
            take.append(len(part[:k - sum(take)]))
        at = np.cumsum(take)
        assert np.array_equal(flat[:at[0]], up[:k]) and (score[b, :at[0]] == np.inf).all()
        if take[1]:
            judge_selection(np.where(np.isfinite(want), want, -1e30).reshape(n, V), flat[at[0]:at[1]], score[b, at[0]:at[1]], take[1], tol=3e-5, margin=2e-5,
                            what="request %d" % b)
        assert np.array_equal(flat[at[1]:at[2]], down[:take[2]]) and (score[b, at[1]:at[2]] == -np.inf).all()
        assert np.array_equal(flat[at[2]:], none[:take[3]]) and np.isnan(score[b, at[2]:]).all()


@pytest.mark.parametrize("high", [0x7FFFFFFF, 0x7FFFFFFC, 0x7F800000, 0x3F800000])
def test_select_cut_spans_all_score_keys(high):
    """Without a bound a request's candidates rank by their score keys, whatever the scores are.  All candidates but one carry the NaN of the lowest
    key, the other one (not among the cut's samples, every second candidate) a score of a far higher key, up to the highest there is."""
    n, k, at = 2048, 5, 1027
    cum = np.full((1, n), 0xFFFFFFFF, np.uint32)
    cum[0, at] = high
    parent, tok, score = (t.cpu().numpy() for t in binding.op_select(torch.zeros(1, n, 1, device="cuda"), torch.from_numpy(cum.view(np.int32)).cuda().view(torch.float32), k))
    assert parent.tolist() == [[at, 0, 1, 2, 3]] and not tok.any()
    assert score.view(np.uint32)[0].tolist() == [high] + [0xFFFFFFFF] * (k - 1)


@pytest.mark.parametrize("dtype,B,d", [("f32", 5, 128), ("bf16", 140, 256)])
def test_request_of_nan_contexts_leaves_the_others_alone(dtype, B, d):
    w = synth.Workload("poisoned", dtype, B, 24, d, 3, 1, 4, 2 * d, 3, [264, 96, 512], [64, 64, 64])
    dec = binding.decoder_for(w, synth.make_weights(w))
    g = torch.Generator(device="cuda").manual_seed(d)
    ctx = torch.randn(B, w.S, d, generator=g, device="cuda").to(binding.torch_dtype(dtype))
    want_sid, want_lp = dec.decode_batch(ctx, None, w.beam)
    ctx[2] = float("nan")
    sid, lp = dec.decode_batch(ctx, None, w.beam)
    torch.cuda.synchronize()
    others = [b for b in range(B) if b != 2]
    assert torch.equal(sid[others], want_sid[others]) and torch.equal(lp[others], want_lp[others])
    V = torch.tensor(w.V, device="cuda")
    assert (sid >= 0).all() and (sid < V).all()
    assert len(torch.unique(sid[2].cpu(), dim=0)) == w.beam[-1]
    dec.close()


# live: tokens that are not masked, fewer and more than k.  Rows that get their own cut because the bound lists them (3 rows per request) and without a bound (9 rows; one row in
# many requests)
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("V,live", [(72, 5), (72, 66), (256, 10), (256, 200), (1024, 12), (1024, 700), (2048, 20), (2048, 1024)])
@pytest.mark.parametrize("B,n,k", [(4, 3, 16), (5, 9, 32), (520, 1, 16)])
def test_select_of_infinite_cumulative_score_over_masked_tokens(B, n, k, V, live, half):
    """Every second request has a row whose cumulative score is +inf: its live tokens score +inf, its masked ones NaN.  The requests between them come out as they do
    beside numbers (rows share workgroups and their LDS)."""
    rng = np.random.default_rng([B, n, V, k, live, half])
    logits = rng.standard_normal((B, n, V)).astype(np.float16 if half else np.float32)
    logits.reshape(B * n, V)[np.arange(B * n)[:, None], np.argsort(rng.random((B * n, V)), axis=1)[:, live:]] = -np.inf
    cum = -6.0 * rng.random((B, n)).astype(np.float32)
    z = torch.from_numpy(logits).cuda()
    plain = [t.cpu().numpy() for t in binding.op_select(z, torch.from_numpy(cum).cuda(), k)]
    cum[::2, n // 2] = np.inf
    print("B n V k live", B, n, V, k, live, "half", half, flush=True)
    got = [t.cpu().numpy() for t in binding.op_select(z, torch.from_numpy(cum).cuda(), k)]
    for g, p in zip(got, plain):
        assert np.array_equal(g[1::2], p[1::2])
    for b in range(0, B, 2):
        flat, score = got[0][b].astype(np.int64) * V + got[1][b], got[2][b]
        assert len(np.unique(flat)) == k and flat.min() >= 0 and flat.max() < n * V
        with np.errstate(invalid="ignore"):
            want = cum[b].astype(np.float64)[:, None] + np.stack([oracle.prim_log_softmax(z) for z in logits[b].astype(np.float32)])
        want = want.ravel()
        parts = [np.flatnonzero(w) for w in (want == np.inf, np.isfinite(want), want == -np.inf, np.isnan(want))]  # (in the order of their ranks)
        at = np.cumsum([0] + [len(p) for p in parts]).clip(max=k)
        for part, lo, hi in zip(parts, at[:-1], at[1:]):
            if part is parts[1] and hi > lo:
                judge_selection(np.where(np.isfinite(want), want, -1e30).reshape(n, V), flat[lo:hi], score[lo:hi], hi - lo, tol=3e-5, margin=2e-5, what="request %d" % b)
            else:  # equal scores go by their tokens
                assert np.array_equal(flat[lo:hi], part[:hi - lo]) and np.array_equal(score[lo:hi], want[part[:hi - lo]].astype(np.float32), equal_nan=True)
