"""Selections of one row in one launch, and of few short rows cut one by one: against a float64 reference over masks, ties and edges of the tiles."""
import numpy as np
import pytest
import torch

from paper_2602_22732_amd import binding

pytestmark = pytest.mark.gpu


def logits(kind, B, n, V, g):
    z = torch.randn(B, n, V, generator=g) * 2
    if kind == "masked":       # half of the tokens
        z[:, :, : V // 2] = -float("inf")
    if kind == "low":          # a finite mask that presses the others together
        z[:, :, : V // 3] = -1e9
    if kind == "tied":         # more equal scores than survive
        z = torch.round(z)
    if kind == "wide":         # scores over some hundreds
        z = z * 40
    return z


# one row: one key per thread, 256 keys and one more (sorted, cut), a piece per thread and more, the block kernel's order (V not a multiple of 4, more than 8192
# tokens), everything survives.  Several: 64 and 65 rows of 1024 keys and of more, all keys of a request sorted and cut, 8192 keys in all and one row more
@pytest.mark.parametrize("B,n,V,k", [(3, 1, 1, 1), (2, 1, 256, 256), (2, 1, 260, 16), (2, 1, 1024, 700), (2, 1, 4096, 1), (2, 1, 4100, 512), (2, 1, 8192, 4096), (2, 1, 5001, 600), (1, 1, 16384, 4096),
                                     (512, 1, 264, 3), (513, 1, 264, 3), (4, 16, 256, 16), (2, 65, 1024, 64), (64, 64, 1024, 64), (3, 3, 2048, 1500), (1, 128, 72, 64), (1, 129, 72, 64),
                                     (2, 4, 8, 8)])
@pytest.mark.parametrize("kind", ["plain", "masked", "low", "tied", "wide"])
def test_short_selections(B, n, V, k, kind):
    g = torch.Generator().manual_seed(B + n * 7 + V + k)
    z, cum = logits(kind, B, n, V, g), -torch.sort(torch.rand(B, n, generator=g) * 6 + 3, dim=1).values
    par, tok, score = binding.op_select(z.cuda(), cum.cuda(), k)
    par, tok, score = par.cpu().numpy(), tok.cpu().numpy(), score.cpu().numpy().astype(np.float64)
    ref = (cum[:, :, None].double() + torch.log_softmax(z.double(), dim=2)).reshape(B, n * V).numpy()
    for b in range(B):
        flat = par[b].astype(np.int64) * V + tok[b]
        assert len(set(flat.tolist())) == k and flat.min() >= 0 and flat.max() < n * V
        order = np.argsort(-ref[b], kind="stable")
        kth = ref[b][order[k - 1]]
        got = ref[b][flat]
        fin = np.isfinite(got)
        # float32 scores: a few roundings of numbers below 32; four half units in the last place of larger ones, of the score or, in wide rows, of the log-sum-exp (about the best logit,
        # up to 200: its own rounding, the difference's and the sum's)
        unit = lambda x: 2.0**-22 * ((np.abs(x) * (np.abs(x) > 32)) + (abs(float(z[b].max())) if kind == "wide" else 0.0))
        assert np.array_equal(fin, np.isfinite(score[b])) and (np.abs(got[fin] - score[b][fin]) <= 1e-5 + unit(got[fin])).all()
        assert (got >= kth - (1e-5 + unit(kth) if np.isfinite(kth) else 0.0)).all() and (np.diff(score[b][fin]) <= 0).all()
        if kind == "low":  # every token that is not masked comes before those that are
            low = z[b].reshape(-1).numpy()[flat] < -1e8
            live = min(k, int((z[b] > -1e8).sum()))
            assert not low[:live].any() and low[live:].all()
        if kind in ("masked", "tied"):  # equal scores go by the lowest (row, token)
            eq = np.flatnonzero(score[b][1:] == score[b][:-1])
            assert (flat[eq + 1] > flat[eq]).all()


# up to 512 (rows of a multiple of 4 tokens, at most 8192) or 256 requests of one row run in one launch, more in two.  nan: a cumulative score and some logits, NaN of either sign
@pytest.mark.parametrize("V,k,most,half", [(V, k, 512, half) for V, k in ((72, 16), (264, 264), (1032, 300), (2048, 64), (2056, 64), (8192, 700)) for half in (False, True)]
                         + [(301, 16, 256, False), (1030, 600, 256, False), (16384, 200, 256, False)])
@pytest.mark.parametrize("kind", ["plain", "masked", "tied", "nan"])
def test_one_launch_selects_what_two_do(V, k, most, kind, half):
    g = torch.Generator().manual_seed(V + k)
    z, cum = logits(kind, 4, 1, V, g), -torch.rand(4, 1, generator=g)
    if kind == "nan":  # (one sign to a row)
        z[0, 0, V // 2] = float("nan")
        z[1, 0, 3] = z[1, 0, V - 2] = -float("nan")
        z[3, 0, 5] = -float("nan")
        cum[:3, 0] = torch.tensor([float("nan"), -float("nan"), float("nan")])
    z, cum = z.cuda().to(torch.float16 if half else torch.float32), cum.cuda()
    one = binding.op_select(z, cum, k)
    two = binding.op_select(z.repeat(most // 4 + 1, 1, 1), cum.repeat(most // 4 + 1, 1), k)
    for a, b in zip(one, two):
        assert torch.equal(a.view(torch.int32), b[-4:].view(torch.int32))


# half-precision rows walked several to a wavefront, the next one requested ahead, as one row to a wavefront: rows that do not fill the last workgroup, two to eight to a wavefront, pieces that
# no or some of the lanes have, every lane (1024; 2048, 4096 and 8192 with as many candidates as leave few wavefronts)
@pytest.mark.parametrize("B,n,V,k", [(331, 101, 264, 150), (1300, 102, 72, 64), (520, 101, 1024, 200), (331, 101, 1032, 140), (1025, 129, 2040, 130), (651, 101, 2056, 256), (400, 170, 4088, 9), (901, 130, 4104, 64), (325, 101, 2048, 1030), (331, 101, 4096, 1300), (331, 101, 8192, 2049),
                                     (331, 101, 4104, 2049)])
def test_many_short_rows_as_few(B, n, V, k):
    g = torch.Generator(device="cuda").manual_seed(V)
    z = torch.randn(B, n, V, generator=g, device="cuda", dtype=torch.float16)
    z[:, 1::2, : V // 2] = -float("inf")
    z[1::3, n - 1] = float("nan")
    cum = -torch.sort(torch.rand(B, n, generator=g, device="cuda") * 6 + 3, dim=1).values
    many = binding.op_select(z, cum, k)
    for lo in (0, B // 2, B - 8):
        few = binding.op_select(z[lo:lo + 8], cum[lo:lo + 8], k)
        for a, b in zip(few, many):
            assert torch.equal(a.view(torch.int32), b[lo:lo + 8].view(torch.int32))
