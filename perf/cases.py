"""What a user of this package has the GPU do, as measurable cases: decodes of a batch of requests through
binding.Decoder.decode_batch, from one request to the benchmark's large batches, and the selection on its own.

A case is a dict of plain values.  listed() names the cases, draw() gives further ones of the same ranges, prepare() makes
what a serving process has in hand before the call (the decoder with its weights, the encoded contexts, the kept workspace and
output buffers), run() is the call, work() the bytes and operations it cannot do without, tolerance() how far another
correct implementation at the same precision may be off.
"""
import math

import torch

from paper_2602_22732_amd import binding

# ---- model shapes -----------------------------------------------------------------------------------------------------
# The shapes of the benchmark configurations (paper_2602_22732_amd/synth.py): d, heads, FFN width, layers, lazy layers, codebooks,
# beam widths.  "mixed" is the large model's width with the published deployment's structure (nine layers, six of them lazy,
# three levels, codebooks of 16k/4k/1k entries, beams that double per level).
MODELS = {
    "tiny": dict(d=128, H=4, F=512, L=2, K=1, V=(256, 256, 256), beam=(16, 16, 16), S=64),
    "small": dict(d=256, H=8, F=1024, L=4, K=2, V=(1024, 1024, 1024), beam=(64, 64, 64), S=256),
    "medium": dict(d=512, H=8, F=2048, L=6, K=4, V=(4096, 4096, 4096), beam=(128, 256, 512), S=512),
    "large": dict(d=1024, H=16, F=4096, L=8, K=6, V=(8192, 8192, 8192, 8192), beam=(256, 512, 512, 1024), S=1024),
    "mixed": dict(d=1024, H=16, F=4096, L=9, K=6, V=(16384, 4096, 1024), beam=(128, 256, 512), S=512),
}


def _decode(name, model, B, S, dtype="bf16", min_len=0, scale=1.0, lazy=-1, value=0, fp8=False, vanilla=False, zipf=False):
    """min_len: shortest context of the batch (lengths uniform in [min_len, S]; 0: all S).  scale: beam scale of this call (the
    load-adaptive schedule).  lazy: lazy layers (-1: the model's).  value: buckets of the value step (0: none).  zipf: popularity
    bias on the classifiers."""
    return {"name": name, "path": "decode", "model": model, "B": B, "S": S, "dtype": dtype, "min_len": min_len, "scale": scale, "lazy": lazy,
            "value": value, "fp8": fp8, "vanilla": vanilla, "zipf": zipf}


def _select(name, B, n, V, k, half):
    return {"name": name, "path": "select", "B": B, "n": n, "V": V, "k": k, "half": half}


def listed():
    return [
        # configuration 1: the smallest decode, float32; every launch is short
        _decode("tiny-f32", "tiny", 4, 64, dtype="f32"),
        # configuration 2: a small model at its batch
        _decode("small", "small", 64, 256),
        # an interactive call: one request of the medium model
        _decode("medium-one", "medium", 1, 512),
        # configuration 3 at its batch
        _decode("medium", "medium", 256, 512),
        # re-ranking traffic: the value step on ragged contexts of an odd length, an odd batch
        _decode("medium-value", "medium", 45, 389, min_len=97, value=256),
        # the plain autoregressive decoder the lazy one is compared with
        _decode("medium-vanilla", "medium", 32, 512, lazy=0, vanilla=True),
        # the deployment's structure: codebooks of different sizes, a mid-size serving batch, popular tokens
        _decode("mixed", "mixed", 32, 500, min_len=125, zipf=True),
        # off-peak traffic on the large model: a handful of requests, full beams
        _decode("large-few", "large", 8, 1024, min_len=256),
        # low-precision inference
        _decode("large-fp8", "large", 128, 1024, min_len=256, fp8=True, zipf=True),
        # peak traffic: the load-adaptive schedule at a quarter of the beams
        _decode("large-peak", "large", 256, 1024, min_len=256, scale=0.25, zipf=True),
        # the benchmark's model and traffic (configuration 5) at half its batch: the largest call
        _decode("large", "large", 1024, 1024, min_len=256, zipf=True),
        # the selection as an operation of its own (callers with logits of their own), half-precision logits
        _select("select", 64, 256, 4096, 512, True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# largest batch a drawn case may have, per model
MOST_B = {"tiny": 64, "small": 256, "medium": 512, "large": 1024, "mixed": 512}


def draw(rng):
    most = work(listed()[10])["flops"]
    while True:
        if rng.random() < 0.12:
            V = 8 * rng.randint(64, 1024) if rng.random() < 0.7 else rng.randint(300, 16384)
            half = V % 8 == 0 and V <= 8192 and rng.random() < 0.6
            n = _log_int(rng, 8, 1024)
            c = _select("", _log_int(rng, 1, 256), n, V, min(_log_int(rng, 16, 1024), n * V), half)
            if 4 * c["B"] * c["n"] * c["V"] > 4 << 30:
                continue
        else:
            model = rng.choice(["tiny", "small", "medium", "medium", "large", "large", "mixed"])
            m = MODELS[model]
            S = _log_int(rng, m["S"] // 4, m["S"])
            if rng.random() < 0.3:
                S = m["S"]
            kind = rng.choice(["plain", "plain", "plain", "value", "vanilla", "lazy", "fp8"])
            dtype = "f32" if model == "tiny" else "bf16"
            if kind == "fp8" and (dtype == "f32" or model == "small"):
                kind = "plain"
            c = _decode("", model, _log_int(rng, 1, MOST_B[model]), S, dtype=dtype,
                        min_len=max(1, S // 4) if rng.random() < 0.6 else 0,
                        scale=rng.choice([0.25, 0.5, 1.0, round(rng.uniform(0.2, 1.0), 2)]),
                        lazy=0 if kind == "vanilla" else rng.randint(0, m["L"] - 1) if kind == "lazy" else -1,
                        value=rng.choice([100, 256, 512]) if kind == "value" else 0,
                        fp8=kind == "fp8", vanilla=kind == "vanilla", zipf=rng.random() < 0.5)
        if work(c)["flops"] <= most and _state_bytes(c) <= 60e9:
            del c["name"]
            return c


# ---- sizes of a case --------------------------------------------------------------------------------------------------
def _shape(case):
    """The model of a decode case with this call's beams: b_t <= b_{t-1} * V_t always holds for these codebooks."""
    m = dict(MODELS[case["model"]])
    m["T"] = len(m["V"])
    m["max_beam"] = list(m["beam"])
    m["beam"] = [max(1, int(round(b * case["scale"]))) for b in m["beam"]]
    if case["lazy"] >= 0:
        m["K"] = case["lazy"]
    m["A"] = m["L"] - m["K"]
    return m


def _mean_len(case):
    return 0.5 * (case["min_len"] + case["S"]) if case["min_len"] else float(case["S"])


def _state_bytes(case):
    """About what prepare() holds: contexts and workspace (the keys and values of the autoregressive layers, the per-row buffers)."""
    if case["path"] == "select":
        return 8.0 * case["B"] * case["n"] * case["V"]
    m = _shape(case)
    e = 4 if case["dtype"] == "f32" else 2
    rows = [1] + m["beam"][:-1] + ([m["beam"][-1]] if case["value"] else [])
    widest = max(rows)
    per_row = m["d"] * (4 + 3 * e) + m["F"] * 2 * e + max(m["V"]) * 4
    return case["B"] * (case["S"] * m["d"] * e * (1 + 3 * m["A"]) + widest * per_row + sum(rows) * m["A"] * 3 * m["d"] * e)


def work(case):
    """Operations (a multiply-add counts two) and bytes one decode cannot do without: the products of the method on the valid
    rows; every weight, every valid context row and every result once."""
    if case["path"] == "select":
        B, n, V, k = case["B"], case["n"], case["V"], case["k"]
        return {"bytes": B * n * V * (2 if case["half"] else 4) + B * n * 4 + B * k * 12, "flops": 3.0 * B * n * V}
    m = _shape(case)
    B, d, F, L, K, A, T, V = case["B"], m["d"], m["F"], m["L"], m["K"], m["A"], m["T"], m["V"]
    e = 4 if case["dtype"] == "f32" else 2
    ln, Ve = _mean_len(case), case["value"]
    rows = [1] + m["beam"][:-1]
    books = list(V)
    if Ve:
        rows, books = rows + [m["beam"][-1]], books + [Ve]
    R, Tp = float(sum(rows)), len(rows)
    flops = A * 4.0 * ln * d * d                                    # keys and values of the context
    flops += Tp * K * (12.0 * d * d + 4.0 * d * F + 4.0 * ln * d)   # lazy pass
    flops += 0.0 if case["vanilla"] else R * 2.0 * d * d            # Fuse
    flops += R * A * (12.0 * d * d + 4.0 * d * F + 4.0 * ln * d)    # autoregressive layers with their cross-attention
    flops += sum(r * A * 4.0 * (t + 1) * d for t, r in enumerate(rows))
    flops += sum(r * 2.0 * d * v for r, v in zip(rows, books))      # classifiers
    weights = L * (8.0 * d * d + 2.0 * d * F) + 2.0 * d * sum(V[:-1]) + V[-1] * d + (V[-1] * d + Ve * d if Ve else 0) + 3.0 * d * d
    out = m["beam"][-1] * (4.0 * T + 4.0 + 4.0 * Ve)
    return {"bytes": weights * e + B * (ln * d * e + out), "flops": B * flops}


def tolerance(case):
    """SIDs are whole values ranked by a score: two candidates whose scores are closer than the arithmetic resolves may change
    places, which "differ" allows for.  Log-probabilities: float32 sums, or what bf16 (E4M3) operands leave in them."""
    if case["path"] == "select" or case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4, "differ": 0.005}
    return {"rel": 1e-2 if case["fp8"] else 5e-3, "max": 0.1, "differ": 0.01}


# ---- inputs -----------------------------------------------------------------------------------------------------------
def _weights(case, m, g):
    """Random-init parameters drawn on the GPU with the distributions of synth.make_weights: Xavier-uniform matrices, N(0,1)
    embeddings and positions, norm gains around one, and, with popular tokens, a Zipf(1.1) logit bias."""
    td = binding.torch_dtype(case["dtype"])
    d, F, V, T = m["d"], m["F"], m["V"], m["T"]

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda").to(td)

    def xavier(out_f, in_f):
        lim = math.sqrt(6.0 / (in_f + out_f))
        return ((torch.rand(out_f, in_f, generator=g, device="cuda") * 2.0 - 1.0) * lim).to(td)

    def gain():
        return (1.0 + 0.1 * torch.randn(d, generator=g, device="cuda")).to(td)

    w = {"pos": normal(T, d), "bos": normal(d), "emb": [normal(V[t], d) for t in range(T - 1)], "w_g": xavier(d, d), "w_f": xavier(d, 2 * d),
         "ln_out": gain(), "cls": [xavier(V[t], d) for t in range(T)], "cls_bias": None, "layers": []}
    for _ in range(m["L"]):
        lw = {}
        for n in binding.LAYER_FIELDS:
            lw[n] = gain() if n.startswith("ln_") else xavier(F, d) if n == "w1" else xavier(d, F) if n == "w2" else xavier(d, d)
        w["layers"].append(lw)
    if case["zipf"]:
        w["cls_bias"] = [-1.1 * torch.log(torch.randperm(V[t], generator=g, device="cuda").float() + 1.0) for t in range(T)]
    if case["value"]:
        w["value_pos"], w["value_emb"], w["value_cls"], w["value_bias"] = normal(d), normal(V[-1], d), xavier(case["value"], d), None
    return w


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["path"] == "select":
        # a level of a decode: logits of all live beams (popular tokens stand out), the beams' running log-probabilities
        B, n, V = case["B"], case["n"], case["V"]
        pop = -1.1 * torch.log(torch.randperm(V, generator=g, device="cuda").float() + 1.0)
        logits = 0.5 * torch.randn(B, n, V, generator=g, device="cuda") + pop
        cum = -torch.sort(torch.rand(B, n, generator=g, device="cuda") * 6.0 + 3.0, dim=1).values
        return {"logits": logits.to(torch.float16 if case["half"] else torch.float32), "cum": cum.contiguous(), "k": case["k"]}
    m = _shape(case)
    B, S = case["B"], case["S"]
    dec = binding.Decoder(m["d"], m["H"], m["F"], m["L"], m["K"], m["T"], m["V"], _weights(case, m, g), case["dtype"], m["max_beam"], B, S,
                          Ve=case["value"], fp8=case["fp8"], vanilla=case["vanilla"])
    ctx = torch.randn(B, S, m["d"], generator=g, device="cuda", dtype=binding.torch_dtype(case["dtype"]))
    ctx_len = None
    if case["min_len"]:
        ctx_len = torch.randint(case["min_len"], S + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    b = m["beam"][-1]
    return {"dec": dec, "ctx": ctx, "ctx_len": ctx_len, "beam": m["beam"],
            "workspace": torch.empty(dec.workspace_bytes(B, S, m["beam"]), dtype=torch.uint8, device="cuda"),
            "out_sid": torch.empty(B, b, m["T"], dtype=torch.int32, device="cuda"),
            "out_logprob": torch.empty(B, b, dtype=torch.float32, device="cuda"),
            "out_value": torch.empty(B, b, case["value"], dtype=torch.float32, device="cuda") if case["value"] else None}


def run(state):
    if "logits" in state:
        parent, tok, score = binding.op_select(state["logits"], state["cum"], state["k"])
        return {"parent": parent, "tok": tok, "score": score}
    value = state["out_value"] is not None
    out = state["dec"].decode_batch(state["ctx"], state["ctx_len"], state["beam"], workspace=state["workspace"], out_sid=state["out_sid"],
                                    out_logprob=state["out_logprob"], value=value, out_value=state["out_value"])
    return {"sid": out[0], "logprob": out[1], "value": out[2]} if value else {"sid": out[0], "logprob": out[1]}
