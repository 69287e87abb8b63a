"""Selections over masked logits: -inf, or masks so low that all other tokens look alike beside them.  The request's bound has to survive
the mask: the rows list about k candidates, where without a bound each would list k of its own."""
import numpy as np
import pytest
import torch

from gpu_common import judge_selection
from paper_2602_22732_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("mask", [[-np.inf], [-1e4], [-65504.0], [-np.inf, -65504.0, -3000.0]])
@pytest.mark.parametrize("B,n,V,k,live", [(3, 5, 264, 64, 100), (2, 130, 4096, 300, 1000), (2, 4, 8192, 700, 2500), (1, 512, 1032, 512, 513)])
def test_masked_logits_keep_the_request_bound(B, n, V, k, live, mask, half):
    rng = np.random.default_rng([B, n, V, k, half])
    logits = rng.standard_normal((B, n, V)).astype(np.float16 if half else np.float32)
    for b in range(B):
        for i in range(n):
            dead = rng.permutation(V)[live:]
            logits[b, i, dead] = rng.choice(mask, len(dead))
    cum = (-2.5 * np.arange(n) - rng.random((B, n))).astype(np.float32)
    z, c = torch.from_numpy(logits).cuda(), torch.from_numpy(cum).cuda()
    L = binding.lib()
    ws = torch.empty(int(L.gr4ad_op_select_workspace_bytes(B, n, V, k)), dtype=torch.uint8, device="cuda")
    parent, tok = (torch.empty(B, k, dtype=torch.int32, device="cuda") for _ in range(2))
    score = torch.empty(B, k, device="cuda")
    entry = L.gr4ad_op_select_f16 if half else L.gr4ad_op_select
    assert entry(z.data_ptr(), c.data_ptr(), B, n, V, k, ws.data_ptr(), ws.numel(), parent.data_ptr(), tok.data_ptr(), score.data_ptr(),
                 torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    m = min(k, V)
    at = (8 * B * n * m + 255) // 256 * 256  # candidates [B][n*m], then how many of them each request listed, min(m, 32) ints apart
    listed = ws[at:].view(torch.int32)[:B * min(m, 32):min(m, 32)].cpu().numpy()
    for b in range(B):
        with np.errstate(divide="ignore"):
            e = np.exp(logits[b].astype(np.float64))
            allsc = cum[b].astype(np.float64)[:, None] + np.log(e / e.sum(1, keepdims=True))
        flat = parent[b].cpu().numpy().astype(np.int64) * V + tok[b].cpu().numpy()
        assert len(np.unique(flat)) == k
        judge_selection(allsc, flat, score[b].cpu().numpy(), k, tol=3e-5, margin=2e-5, what="request %d" % b)
        assert k <= listed[b] <= 2 * k, listed
