"""Selections whose request bound comes from several rows (one more power of two of rows per 64 beams), on both logit types."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import judge_selection
from paper_2602_22732_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("spread", ["level", "steep", "best_row_last", "equal_logits"])
@pytest.mark.parametrize("B,n,V,k", [(3, 1, 1024, 7), (2, 127, 264, 64), (2, 128, 264, 65), (1, 512, 1032, 1032), (1, 2048, 64, 60)])
def test_select_bound_from_several_rows(B, n, V, k, spread, half):
    rng = np.random.default_rng([B, n, V, k, half])
    logits = rng.standard_normal((B, n, V)).astype(np.float16 if half else np.float32)
    if spread == "equal_logits":
        logits[:] = 0.25
    cum = (-3.0 - 0.02 * rng.random((B, n))).astype(np.float32)
    if spread == "steep":
        cum -= 2.5 * np.arange(n, dtype=np.float32)
    if spread == "best_row_last":
        cum[:, :-1] -= 4.0
    parent, tok, score = (t.cpu().numpy() for t in binding.op_select(torch.from_numpy(logits).cuda(), torch.from_numpy(cum).cuda(), k))
    for b in range(B):
        allsc = cum[b].astype(np.float64)[:, None] + np.stack([oracle.prim_log_softmax(logits[b, i].astype(np.float32)) for i in range(n)])
        flat = parent[b].astype(np.int64) * V + tok[b]
        assert len(np.unique(flat)) == k
        judge_selection(allsc, flat, score[b], k, tol=3e-5, margin=2e-5, what="select b=%d" % b)


@pytest.mark.parametrize("V", [4104, 8192])
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("B,n", [(4, 2048), (8193, 1), (2049, 4)])  # 8192 rows, whose own cuts run on wavefronts alone on their SIMD, and more, which share
def test_select_lists_many_wide_rows(B, n, V, half):
    """Equal scores overflow every row's segment, so that all rows get their own cut: the k lowest tokens of the request's first row."""
    k = 24
    logits = torch.full((B, n, V), 0.25, dtype=torch.float16 if half else torch.float32, device="cuda")
    logits[:, -1, V - 3] = 1.0
    parent, tok, score = binding.op_select(logits, torch.zeros(B, n, device="cuda"), k)
    rest = torch.arange(k - 1, dtype=torch.int32, device="cuda")
    assert (parent[:, 0] == n - 1).all() and (tok[:, 0] == V - 3).all()
    assert (parent[:, 1:] == 0).all() and (tok[:, 1:] == rest).all()
    lse_last, lse = (np.log((V - 1) * np.exp(0.25) + np.exp(1.0)), 0.25 + np.log(V))
    np.testing.assert_allclose(score[:, 0].double().cpu().numpy(), 1.0 - lse_last, atol=2e-5)
    np.testing.assert_allclose(score[:, 1:].double().cpu().numpy(), 0.25 - (lse_last if n == 1 else lse), atol=2e-5)


# n * V candidates (V <= k: rows are not cut): kept in registers up to 8192 and read twice above, in pairs or one by one (odd segments of the
# second request); the cut's bin holds few keys, hundreds of equal ones ("levels"), or nearly all of them beside far ones ("far")
@pytest.mark.parametrize("spread", ["level", "levels", "far"])
@pytest.mark.parametrize("n,V,k", [(147, 7, 7), (130, 8, 512), (129, 8, 513), (1024, 8, 2048), (1024, 8, 2049), (911, 9, 64), (1025, 8, 1024), (1025, 8, 4096)])
def test_select_cuts_a_request(n, V, k, spread):
    B = 2
    rng = np.random.default_rng([n, V, k])
    logits = rng.standard_normal((B, n, V)).astype(np.float32)
    cum = (-3.0 - 0.02 * rng.random((B, n))).astype(np.float32)
    if spread == "levels":
        logits[:] = 0.25
        cum = (-3.0 - rng.integers(0, 3, (B, n))).astype(np.float32)
    if spread == "far":
        cum[:, ::7] = -1e30
    parent, tok, score = (t.cpu().numpy() for t in binding.op_select(torch.from_numpy(logits).cuda(), torch.from_numpy(cum).cuda(), k))
    for b in range(B):
        allsc = cum[b].astype(np.float64)[:, None] + np.stack([oracle.prim_log_softmax(logits[b, i]) for i in range(n)])
        flat = parent[b].astype(np.int64) * V + tok[b]
        assert len(np.unique(flat)) == k
        assert np.all((score[b][:-1] > score[b][1:]) | ((score[b][:-1] == score[b][1:]) & (flat[:-1] < flat[1:])))
        judge_selection(allsc, flat, score[b], k, tol=3e-5, margin=2e-5, what="select b=%d" % b)
