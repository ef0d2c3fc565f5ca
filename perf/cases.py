"""Timed cases of the token-pruning path: what a serving program has this library do, over the range it is used in.

Three kinds of pass, each through the entry points a caller uses:
  prompt  scores of a prompt's tokens (vatp_prefill_score, vatp_prefill_score_lse, vatp_prefill_score_window);
  prune   the prompt's cache cut to its budget (vatp_select_compact);
  decode  one generated token through a run of layers, each layer's cache appended to, scored and cut back to its
          budget (PrunedKVCache.decode_prune_step).
A case holds the sizes: `length` is the prompt's length (the longest one where `ragged`), `budget_pct` the share of it
that stays, `group` the query heads per K/V head, `window` the history window in steps (-1: accumulated scores).
Sizes are those of the named workloads of the benchmark, or lie between them.
"""
import math

import torch

import paper_2406_12335_amd as vatp
from paper_2406_12335_amd.runner import PrunedKVCache

_DTYPES = {"fp32": torch.float32, "bf16": torch.bfloat16}
_BASE = dict(batch=1, heads=32, group=1, head_dim=128, dtype="bf16", length=4096, ragged=False, sinks=2, recent=64,
             sigma=0.5, budget_pct=50, window=-1, lse=False, attend=False, layers=1)


def _case(kind, name=None, **sizes):
    case = dict(_BASE, kind=kind, **sizes)
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # a short prompt on a small fp32 model: the smallest call, all launch and latency
        _case("prompt", "prompt_tiny", heads=4, head_dim=64, dtype="fp32", length=256, recent=16),
        # one layer of a 7B-shaped model, one request of ordinary length
        _case("prompt", "prompt_layer"),
        # a batch of requests of unequal length, one layer of the same model
        _case("prompt", "prompt_ragged16", batch=16, length=8192, ragged=True, budget_pct=30),
        # a long document, one layer of the same model: the largest call
        _case("prompt", "prompt_long32k", length=32768, sinks=4, sigma=1.0, recent=128, budget_pct=10),
        # grouped-query model behind a fused attention kernel, which hands over its row log-sum-exps
        _case("prompt", "prompt_gqa_lse", batch=8, heads=8, group=4, lse=True, length=4001),
        # scores over a history window of 400 steps instead of accumulated ones
        _case("prompt", "prompt_window400", window=400),
        # a batch on a model with heads of 64
        _case("prompt", "prompt_heads_of_64", batch=4, heads=16, head_dim=64, length=2048),
        # the prompt of a batch of 8 cut to a fifth, one layer
        _case("prune", "prune_batch8", batch=8, budget_pct=20),
        # one token on the small fp32 model
        _case("decode", "decode_tiny", heads=4, head_dim=64, dtype="fp32", length=256, recent=16),
        # one token of a single request, with the attention output of the layer
        _case("decode", "decode_layer", attend=True),
        # one token of a batch of 8 through 8 consecutive layers of the 32 (a pipeline stage): together they are
        # far larger than the last-level cache
        _case("decode", "decode_batch8_stack", batch=8, budget_pct=20, layers=8),
        # one token of a batch of requests of unequal length on a grouped-query model, with the attention output
        _case("decode", "decode_ragged16_gqa", batch=16, heads=8, group=4, length=8192, ragged=True, budget_pct=30,
              attend=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prompt", "prompt", "prompt", "prune", "decode", "decode", "decode"])
    dtype, head_dim = rng.choice([("bf16", 128)] * 5 + [("bf16", 64)] * 2 + [("fp32", 64), ("fp32", 128)])
    group = rng.choice([1, 1, 1, 2, 4, 8]) if kind != "prune" else 1
    heads = rng.choice([1, 2, 4, 5, 8, 12, 16, 20, 32, 40])
    if group > 1:
        heads = rng.choice([1, 2, 4, 8])
    batch = rng.choice([1, 1, 2, 3, 4, 6, 8, 11, 16])
    length = _log_uniform(rng, 100, 32768)
    recent = rng.choice([16, 32, 64, 128])
    recent = min(recent, length // 8)
    window = rng.choice([-1, -1, -1, 100, 400]) if kind != "prune" else -1
    window = min(window, length - 1)
    lse = kind == "prompt" and window < 0 and length <= 8192 and rng.random() < 0.2
    case = _case(kind, batch=batch, heads=heads, group=group, head_dim=head_dim, dtype=dtype, length=length,
                 ragged=batch > 1 and window < 0 and rng.random() < 0.5, sinks=rng.choice([0, 2, 4]), recent=recent,
                 sigma=rng.choice([0.5, 1.0]), budget_pct=rng.choice([20, 30, 50, 70]), window=window, lse=lse,
                 attend=kind == "decode" and rng.random() < 0.5, layers=rng.choice([1, 1, 2, 4]) if kind == "decode" else 1)
    # no case larger than the listed ones: half the batch, then half the heads, then half the length
    while _too_large(case):
        for field, least in (("layers", 1), ("batch", 1), ("heads", 4), ("length", 100)):
            if case[field] > least:
                case[field] = max(least, case[field] // 2)
                break
    case["recent"] = min(case["recent"], case["length"] // 8)
    case["window"] = min(case["window"], case["length"] - 1)
    case["ragged"] = case["ragged"] and case["batch"] > 1
    return case


def _too_large(case):
    rows = case["batch"] * case["heads"] * case["length"]
    row_bytes = case["head_dim"] * (2 if case["dtype"] == "bf16" else 4)
    if case["kind"] == "prompt":
        # (fp32 products have a sixteenth of the rate of bf16 ones; attention rows of a window are stored)
        flops = _pairs(case, [case["length"]] * case["batch"]) * case["heads"] * case["group"] * 2 * case["head_dim"]
        hist = rows * (case["window"] + 1) * 4 if case["window"] >= 0 else 0
        most = 4.4e12 if case["dtype"] == "bf16" and case["head_dim"] == 128 else 7e10
        return flops > most or hist > 1 << 30 or rows * (2 + case["group"]) * row_bytes > 6 << 30
    if case["kind"] == "prune":
        return rows * row_bytes > 3 << 29
    kept = rows * case["layers"] * case["budget_pct"] // 100
    hist = kept * (case["window"] + 2) * 4 if case["window"] >= 0 else 0
    return kept * row_bytes > 1 << 29 or hist > 1 << 31


def _lens(case, seed):
    """Prompt lengths: the nominal one, or spread evenly between an eighth of it and all of it."""
    if not case["ragged"]:
        return [case["length"]] * case["batch"]
    gen = torch.Generator()
    gen.manual_seed(seed)
    lo = max(case["length"] // 8, case["recent"] + case["sinks"] + 1)
    spread = case["length"] - lo
    n = case["batch"]
    order = torch.randperm(n, generator=gen).tolist()      # (the same lengths for every seed, dealt out differently)
    return [lo + spread * order[b] // max(1, n - 1) for b in range(n)]


def _budgets(case, lens):
    return [min(L, max(L * case["budget_pct"] // 100, case["sinks"] + case["recent"])) for L in lens]


class _Draws:
    """Random tensors on the GPU from one seed."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.gen, device="cuda")

    def uniform(self, *shape):
        return torch.rand(*shape, generator=self.gen, device="cuda")


def _rows(case, draws, cap):
    """K and V rows of a layer and the direction its queries share: leading sinks that every query attends to and
    whose values are near zero, lognormal value norms elsewhere."""
    b, h, g, d, F = case["batch"], case["heads"], case["group"], case["head_dim"], case["sinks"]
    u = draws.normal(b, h, g, d)
    u = 4 * u / u.norm(dim=-1, keepdim=True)
    K = draws.normal(b, h, cap, d)
    if F:
        mean = u.mean(dim=2, keepdim=True)
        K[:, :, :F] = 8 * math.sqrt(d) * mean / (mean * mean).sum(-1, keepdim=True)
    K = K.to(_DTYPES[case["dtype"]])
    V = draws.normal(b, h, cap, d)
    scale = torch.exp(case["sigma"] * draws.normal(b, h, cap, 1))
    scale[:, :, :F] = 0.01
    return u, K, V.mul_(scale).to(_DTYPES[case["dtype"]])


def _attention_received(case, draws, pos, lens):
    """Accumulated attention of the tokens at `pos` after the prompt: about ln(L / i), the sinks far more."""
    L = torch.tensor(lens, device="cuda").view(-1, 1, 1).float()
    S = torch.log(L / (pos.float() + 1)).clamp_(min=0) * torch.exp(0.5 * draws.normal(*pos.shape)) + 1 / L
    return torch.where(pos < case["sinks"], 0.2 * L + S, S)


def _row_lse(case, Q, K, lens):
    """Natural-log row log-sum-exps of the causal softmax, in fp32, as an attention kernel returns them."""
    b, h, g, d = case["batch"], case["heads"], case["group"], case["head_dim"]
    cap = K.shape[2]
    out = torch.zeros(b, h * g, cap, device="cuda")
    ahead = torch.ones(cap, cap, dtype=torch.bool, device="cuda").triu_(1)
    for i in range(b):
        n = lens[i]
        for j in range(h):
            t = Q[i, j * g:(j + 1) * g, :n].float().reshape(g * n, d) @ K[i, j, :n].float().t()
            t = (t.view(g, n, n) / math.sqrt(d)).masked_fill_(ahead[:n, :n], -math.inf)
            out[i, j * g:(j + 1) * g, :n] = torch.logsumexp(t, dim=-1)
    return out


def _params(case, lens, budgets, cap, cap_out=0):
    return vatp.Params(case["batch"], case["heads"], case["head_dim"], _DTYPES[case["dtype"]], case["sinks"],
                       case["recent"], cap, lens, budgets, cap_out=cap_out, q_per_kv=case["group"])


def _prepare_prompt(case, seed):
    b, h, g, d, w = case["batch"], case["heads"], case["group"], case["head_dim"], case["window"]
    draws, lens = _Draws(seed), _lens(case, seed)
    cap = max(lens)
    u, K, V = _rows(case, draws, cap)
    Q = (draws.normal(b, h * g, cap, d).view(b, h, g, cap, d) + u.unsqueeze(3)).to(K.dtype).view(b, h * g, cap, d)
    p = _params(case, lens, _budgets(case, lens), cap)
    ctx = vatp.vatp_create(torch.cuda.current_device())
    call = vatp.binding.CALL_PREFILL_SCORE if w < 0 else vatp.binding.CALL_PREFILL_SCORE_WINDOW
    state = dict(kind="prompt", ctx=ctx, p=p, Q=Q, K=K, V=V, window=w,
                 S=torch.zeros(b, h, cap, device="cuda"), nrm=torch.zeros(b, h, cap, device="cuda"),
                 ws=torch.empty(vatp.vatp_workspace_bytes(ctx, p, call), dtype=torch.uint8, device="cuda"))
    if case["lse"]:
        state["lse"] = _row_lse(case, Q, K, lens)
    if w >= 0:
        state["hist"] = torch.zeros(b, h, w + 1, cap, device="cuda")
    return state


def _prepare_prune(case, seed):
    b, h, d = case["batch"], case["heads"], case["head_dim"]
    draws, lens = _Draws(seed), _lens(case, seed)
    budgets, cap = _budgets(case, lens), max(lens)
    cap_out = max(budgets) + 1
    _, K, V = _rows(case, draws, cap)
    pos = torch.arange(cap, dtype=torch.int32, device="cuda").expand(b, h, cap).contiguous()
    S = _attention_received(case, draws, pos, lens)
    new = lambda *shape, **kw: torch.zeros(b, h, cap_out, *shape, device="cuda", **kw)
    return dict(kind="prune", ctx=vatp.vatp_create(torch.cuda.current_device()), p=_params(case, lens, budgets, cap, cap_out),
                K=K, V=V, S=S, nrm=V.float().abs().sum(-1), pos=pos,
                outs=(new(d, dtype=K.dtype), new(d, dtype=K.dtype), new(), new(), new(dtype=torch.int32),
                      new(dtype=torch.int32)))


def _kept_positions(case, draws, lens, budgets, cap):
    """Which prompt tokens each head's cache holds: sinks, recent window and a random choice of the rest, ascending."""
    b, h, F, R = case["batch"], case["heads"], case["sinks"], case["recent"]
    pos = torch.zeros(b, h, cap, dtype=torch.int64, device="cuda")
    for i, (L, B) in enumerate(zip(lens, budgets)):
        pos[i, :, :F] = torch.arange(F, device="cuda")
        pos[i, :, B - R:B] = torch.arange(L - R, L, device="cuda")
        if B > F + R:
            heavy = draws.uniform(h, L - F - R).topk(B - F - R, dim=-1).indices
            pos[i, :, F:B - R] = F + heavy.sort(dim=-1).values
    return pos


def _prepare_decode(case, seed):
    b, h, g, d, w = case["batch"], case["heads"], case["group"], case["head_dim"], case["window"]
    draws, lens = _Draws(seed), _lens(case, seed)
    budgets = _budgets(case, lens)
    cap, tokens = max(budgets) + 1, 8
    ctx = vatp.vatp_create(torch.cuda.current_device())
    caches, steps = [], []
    held = torch.arange(cap, device="cuda") < torch.tensor(budgets, device="cuda").view(b, 1, 1)
    for _ in range(case["layers"]):
        u, K, V = _rows(case, draws, cap)
        c = PrunedKVCache(b, h, d, K.dtype, case["sinks"], case["recent"], budgets, "cuda:0", cap_cache=cap, ctx=ctx,
                          window=w if w >= 0 else None, q_per_kv=g)
        for name in ("K", "V", "S", "nrm", "pos"):
            for t in getattr(c, name):
                t.zero_()
        c.kept_idx.zero_()
        pos = _kept_positions(case, draws, lens, budgets, cap)
        c.pos[0].copy_(torch.where(held, pos, 0))
        c.K[0].copy_(K.masked_fill_(~held.unsqueeze(-1), 0))
        c.V[0].copy_(V.masked_fill_(~held.unsqueeze(-1), 0))
        c.nrm[0].copy_(c.V[0].float().abs().sum(-1))
        if w < 0:
            # (what was kept of the prompt's middle was kept for its score)
            ages = torch.arange(cap, device="cuda").expand(b, h, cap)
            recent = ages >= torch.tensor(budgets, device="cuda").view(b, 1, 1) - case["recent"]
            S = _attention_received(case, draws, pos, lens)
            c.S[0].copy_(torch.where(held, torch.where(recent, S, S + 0.5), 0))
        else:
            # ring of the last w + 1 steps' attention weights, and the scores as their sums
            rows = w + 2
            for i, L in enumerate(lens):
                j = torch.arange(L - 1 - w, L, device="cuda")
                weight = torch.exp(draws.normal(h, w + 1, cap)) / budgets[i]
                weight[:, :, :case["sinks"]] *= 20
                weight.masked_fill_((pos[i].unsqueeze(1) > j.view(1, -1, 1)) | ~held[i].unsqueeze(1), 0)
                c.hist[i].index_copy_(1, j % rows, weight)
            total = c.hist.double().sum(dim=2)
            c.S[0].copy_(total)
            c.S_lo[0].copy_(total - c.S[0].double())
            c.hid[0].copy_(torch.arange(cap, device="cuda"))
            c.free[c.synced_cur].copy_(torch.tensor(budgets, device="cuda").repeat_interleave(h))
        c.lens = list(budgets)
        caches.append(c)
        q = (draws.normal(tokens, b, h, g, d) + u.unsqueeze(0)).to(K.dtype).view(tokens, b, h * g, d)
        k = draws.normal(tokens, b, h, d).to(K.dtype)
        v = (draws.normal(tokens, b, h, d) * torch.exp(case["sigma"] * draws.normal(tokens, b, h, 1))).to(K.dtype)
        steps.append([(q[t], k[t], v[t]) for t in range(tokens)])
    outs = [torch.zeros(b, h * g, d, device="cuda") if case["attend"] else None for _ in caches]
    return dict(kind="decode", ctx=ctx, caches=caches, steps=steps, outs=outs, next_pos=list(lens), token=0)


def prepare(case, seed):
    return {"prompt": _prepare_prompt, "prune": _prepare_prune, "decode": _prepare_decode}[case["kind"]](case, seed)


def _run_decode(s):
    token = s["token"] % len(s["steps"][0])
    for c, step, out in zip(s["caches"], s["steps"], s["outs"]):
        q, k, v = step[token]
        c.decode_prune_step(q, k, v, s["next_pos"], out=out)
    s["token"] += 1
    s["next_pos"] = [p + 1 for p in s["next_pos"]]
    result = []
    for c, out in zip(s["caches"], s["outs"]):
        i = c.cur
        result.append((c.K[i], c.V[i], c.S[i], c.nrm[i], c.pos[i], c.kept_idx, out))
    return result


def run(s):
    if s["kind"] == "decode":
        return _run_decode(s)
    if s["kind"] == "prune":
        vatp.vatp_select_compact(s["ctx"], s["p"], s["K"], s["V"], s["S"], s["nrm"], s["pos"], *s["outs"])
        return s["outs"]
    if s["window"] >= 0:
        vatp.vatp_prefill_score_window(s["ctx"], s["p"], s["Q"], s["K"], s["V"], s["window"], s["S"], s["nrm"], s["hist"],
                                       s["ws"])
        return s["S"], s["nrm"], s["hist"]
    if "lse" in s:
        vatp.vatp_prefill_score_lse(s["ctx"], s["p"], s["Q"], s["K"], s["V"], s["lse"], s["S"], s["nrm"], s["ws"])
    else:
        vatp.vatp_prefill_score(s["ctx"], s["p"], s["Q"], s["K"], s["V"], s["S"], s["nrm"], s["ws"])
    return s["S"], s["nrm"]


def _pairs(case, lens):
    """(query, key <= query) pairs per query head that count."""
    first = [max(0, L - 1 - case["window"]) if case["window"] >= 0 else 0 for L in lens]
    return sum((L * (L + 1) - f * (f + 1)) // 2 for L, f in zip(lens, first))


def work(case):
    lens = _lens(case, 0)
    budgets = _budgets(case, lens)
    h, g, d, w = case["heads"], case["group"], case["head_dim"], case["window"]
    row = d * (2 if case["dtype"] == "bf16" else 4)
    if case["kind"] == "prompt":
        # one contraction: that the logits are formed twice instead of being stored is this implementation's choice
        queries = [min(L, w + 1) if w >= 0 else L for L in lens]
        data = sum(2 * L * row + g * n * row + 8 * L + (4 * g * L if case["lse"] else 0) + (4 * n * L if w >= 0 else 0)
                   for L, n in zip(lens, queries))
        return {"bytes": h * data, "flops": h * g * 2 * d * _pairs(case, lens)}
    if case["kind"] == "prune":
        return {"bytes": h * sum(8 * L + 4 * B + 4 * row * B + 24 * B for L, B in zip(lens, budgets)), "flops": 0}
    # K once (with the attention output V too), S and nrm read, scores and kept indices written, the recent window's
    # rows moved; with a history window the weight that leaves and the new one, per row
    data = 0
    for B in budgets:
        n, moved = B + 1, case["recent"]
        data += n * row * (2 if case["attend"] else 1) + 8 * n + 8 * B + moved * (4 * row + 16)
        data += 20 * n if w >= 0 else 0
    flops = sum(2 * d * (B + 1) * g * (2 if case["attend"] else 1) for B in budgets)
    return {"bytes": h * case["layers"] * data, "flops": h * case["layers"] * flops}


def tolerance(case):
    if case["kind"] == "prune":
        return "exact"
    # fp32 sums of exponentials and products: against float64 on the same inputs the largest seen are 5e-7 (2-norm) and
    # 1.4e-6 (one component of an attention output)
    return {"rel": 2e-6, "max": 6e-6}
