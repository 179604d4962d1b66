"""Performance cases of the router-gated prefill and decode: what a program that uses this framework has it do.

Kinds of case
  generate     a prompt pass followed by decode steps on a small model: latency and launches
  decode       decode steps of one sequence, or of a batch with a mask of its own each, after a prompt pass
  prefill      first_prefill_route on one prompt or on a batch of prompts of different lengths
  soft         the soft-skip forward with its loss terms (router training)
  lora         merging (and unmerging) one layer's adapters into its seven matrices
  sample       the paper's top-k draw on a batch of logits

Models are the geometries that the benchmark names (LLaMA-3 8B, 3B and 1B class, and the small fp32 one), with fewer
layers where the whole depth would only repeat the same work.  Weights, prompts, routers and masks are drawn from the seed
as the benchmark draws them: N(0, 0.02^2) weights, uniform token ids, the first and the last layer always kept.  The steps
of a decode case are fed given tokens, so that one tie cannot change all that follows, and every pass starts from the
prompt's end; a generate case runs free, as a program that answers does.
"""
import math
import random
from types import SimpleNamespace

import torch

import paper_2410_12513_amd as P

DEV = "cuda"

# layers of the whole model, d_model, query heads, KV heads, head dim, d_ffn, vocabulary, storage type
MODELS = {
    "tiny": (4, 256, 4, 4, 64, 688, 1024, "fp32"),
    "1b": (16, 2048, 32, 8, 64, 8192, 32000, "bf16"),
    "3b": (28, 3072, 24, 8, 128, 8192, 128256, "bf16"),
    "8b": (32, 4096, 32, 8, 128, 14336, 128256, "bf16"),
}


_STREAMS = []


def _stream():
    """The one stream that all models of this program run on: a decode step can be one kernel that needs the whole chip, and two
    such kernels are not run side by side."""
    if not _STREAMS:
        _STREAMS.append(torch.cuda.Stream())
    return _STREAMS[0]


def _desc(case):
    L, D, hq, hkv, hd, f, v, dt = MODELS[case["model"]]
    return SimpleNamespace(n_layers=case.get("layers", L), d_model=D, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ffn=f,
                           vocab=v, dtype=dt, rope_base=10000.0, rms_eps=1e-5)


def _lens(case):
    """Prompt lengths: part of the case, spread over [lo, hi] on a logarithmic scale."""
    rng = random.Random(case["lens_seed"] if "lens_seed" in case else 0)
    lo, hi = case["lo"], case["hi"]
    return [hi if lo == hi else int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) for _ in range(case["batch"])]


def _masks(case):
    """Keep masks, one a sequence: part of the case.  skip_lo .. skip_hi interior layers of each sequence are skipped."""
    rng = random.Random(1 + case.get("mask_seed", 0))
    L, masks = _desc(case).n_layers, []
    for _ in range(case["batch"]):
        k = rng.randint(case["skip_lo"], case["skip_hi"])
        out = set(rng.sample(range(1, L - 1), k)) if k else set()
        masks.append([0 if i in out else 1 for i in range(L)])
    return [masks[0]] * case["batch"] if case.get("same_mask") else masks


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # the small full-precision model, prompt and answer: a call whose cost is launches and latency
        dict(name="generate_tiny_fp32", kind="generate", model="tiny", batch=1, lo=32, hi=32, steps=16, skip_lo=2, skip_hi=2),
        # single-sequence decode, the paper's measure (time per output token), on three model sizes
        dict(name="decode_1b", kind="decode", model="1b", batch=1, lo=512, hi=512, steps=8, skip_lo=4, skip_hi=4),
        dict(name="decode_3b_sampled", kind="decode", model="3b", batch=1, lo=333, hi=333, steps=8, skip_lo=7, skip_hi=7, top_k=10),
        dict(name="decode_8b", kind="decode", model="8b", batch=1, lo=1024, hi=1024, steps=8, skip_lo=8, skip_hi=8),
        # serving: sixteen sequences of different lengths, each with its own mask
        dict(name="decode_8b_batch16", kind="decode", model="8b", layers=8, batch=16, lo=256, hi=2048, steps=8, skip_lo=0, skip_hi=4),
        # long documents: four sequences at 16 k tokens that skip the same layers
        dict(name="decode_8b_batch4_16k", kind="decode", model="8b", layers=4, batch=4, lo=16384, hi=16384, steps=8, skip_lo=1,
             skip_hi=1, same_mask=True),
        # prompts: the benchmark's, a batch of short questions, a long document
        dict(name="prefill_8b_1024", kind="prefill", model="8b", layers=8, batch=1, lo=1024, hi=1024),
        dict(name="prefill_3b_short_batch", kind="prefill", model="3b", layers=8, batch=8, lo=20, hi=300),
        dict(name="prefill_8b_16k", kind="prefill", model="8b", layers=2, batch=1, lo=16384, hi=16384),
        # router training: soft-skip forward and loss terms of a small ragged batch
        dict(name="soft_forward_1b", kind="soft", model="1b", batch=4, lo=100, hi=700),
        # switching an adapter on or off in one layer of the 8B model
        dict(name="lora_8b_layer", kind="lora", model="8b", rank=8, dtype="bf16"),
        # one draw for a batch: the smallest call
        dict(name="sample_batch16", kind="sample", batch=16, vocab=128256, top_k=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: no larger in work than the largest listed one."""
    kind = rng.choice(["generate", "decode", "decode", "decode_batch", "decode_batch", "prefill", "prefill", "prefill", "soft", "lora", "sample"])
    seeds = dict(lens_seed=rng.randrange(1 << 20), mask_seed=rng.randrange(1 << 20))
    if kind == "generate":
        n = _log_int(rng, 3, 200)
        k = rng.randint(0, 2)
        return dict(kind="generate", model="tiny", batch=rng.choice([1, 1, 2]), lo=n, hi=n, steps=rng.randint(4, 16), skip_lo=k, skip_hi=k, **seeds)
    if kind == "decode":
        model = rng.choice(["1b", "3b", "8b"])
        L = rng.randint(4, MODELS[model][0])
        n = _log_int(rng, 16, 4096)
        k = rng.randint(0, L // 2 - 1)
        c = dict(kind="decode", model=model, layers=L, batch=1, lo=n, hi=n, steps=8, skip_lo=k, skip_hi=k, **seeds)
        if rng.random() < 0.4:
            c["top_k"] = rng.choice([1, 5, 10, 40])
        return c
    if kind == "decode_batch":
        model = rng.choice(["1b", "3b", "8b", "8b"])
        L = rng.randint(3, 8)
        lo = _log_int(rng, 32, 4096)
        B = rng.randint(2, 16)
        return dict(kind="decode", model=model, layers=L, batch=B, lo=lo, hi=_log_int(rng, lo, 4096), steps=8, skip_lo=0, skip_hi=L // 2 - 1,
                    same_mask=rng.random() < 0.3, **seeds)
    if kind == "prefill":
        model = rng.choice(["1b", "3b", "8b"])
        L = rng.randint(2, 8)
        B = rng.choice([1, 1, 2, rng.randint(3, 16)])
        hi = _log_int(rng, 16, 16384 if B * L <= 2 else max(64, min(8192, 16384 // (B * max(1, L // 2)))))
        return dict(kind="prefill", model=model, layers=L, batch=B, lo=max(5, int(hi * rng.uniform(0.1, 1.0))), hi=hi, **seeds)
    if kind == "soft":
        model = rng.choice(["1b", "3b", "8b"])
        hi = _log_int(rng, 32, 1500)
        return dict(kind="soft", model=model, layers=rng.randint(2, 6), batch=rng.randint(1, 4), lo=max(5, int(hi * rng.uniform(0.1, 1.0))), hi=hi, **seeds)
    if kind == "lora":
        return dict(kind="lora", model=rng.choice(["1b", "3b", "8b"]), rank=rng.choice([1, 4, 8, 8, 13, 16, 32]), dtype=rng.choice(["bf16", "bf16", "fp32"]))
    return dict(kind="sample", batch=_log_int(rng, 1, 64), vocab=rng.choice([1024, 32000, 50257, 128256]), top_k=rng.choice([1, 5, 10, 20]))


# ------------------------------------------------------------------------------------------------ inputs
def _normal(gen, shape, std, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=gen)


def _weights(d, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1000 + seed)
    dt = torch.bfloat16 if d.dtype == "bf16" else torch.float32
    nq, nkv, D, F = d.n_q_heads * d.head_dim, d.n_kv_heads * d.head_dim, d.d_model, d.d_ffn
    gain = lambda: 1.0 + _normal(gen, (D,), 0.1, torch.float32)  # noqa: E731
    w = {"embed": _normal(gen, (d.vocab, D), 0.02, dt), "lm_head": _normal(gen, (d.vocab, D), 0.02, dt), "final_norm": gain(), "layers": []}
    for _ in range(d.n_layers):
        lw = {"attn_norm": gain(), "mlp_norm": gain()}
        for name, n, k in (("wq", nq, D), ("wk", nkv, D), ("wv", nkv, D), ("wo", D, nq), ("w_gate", F, D), ("w_up", F, D), ("w_down", D, F)):
            lw[name] = _normal(gen, (n, k), 0.02, dt)
        w["layers"].append(lw)
    return w, _normal(gen, (d.n_layers, D), 0.02, torch.float32)


def _tokens(d, n, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3000 + seed)
    return torch.randint(0, d.vocab, (n,), generator=gen, device=DEV, dtype=torch.int32)


LORA_MATRICES = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")


def _lora_shapes(case):
    d = _desc(case)
    nq, nkv = d.n_q_heads * d.head_dim, d.n_kv_heads * d.head_dim
    return dict(wq=(nq, d.d_model), wk=(nkv, d.d_model), wv=(nkv, d.d_model), wo=(d.d_model, nq), w_gate=(d.d_ffn, d.d_model),
                w_up=(d.d_ffn, d.d_model), w_down=(d.d_model, d.d_ffn))


def _lora_inputs(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5000 + seed)
    dt, r = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32, case["rank"]
    return {k: (_normal(gen, (n, m), 0.02, dt), _normal(gen, (r, m), 0.02, torch.float32), _normal(gen, (n, r), 0.01, torch.float32))
            for k, (n, m) in _lora_shapes(case).items()}


def _sample_inputs(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(6000 + seed)
    logits = _normal(gen, (case["batch"], case["vocab"]), 1.3, torch.float32)
    return logits, torch.rand((case["batch"],), generator=gen, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "lora":
        return SimpleNamespace(case=case, mats=_lora_inputs(case, seed), sign=1.0)
    if kind == "sample":
        logits, u = _sample_inputs(case, seed)
        return SimpleNamespace(case=case, logits=logits, u=u, token=torch.zeros(case["batch"], dtype=torch.int32, device=DEV),
                               cand=torch.zeros((case["batch"], case["top_k"]), dtype=torch.int32, device=DEV))
    d, lens, B = _desc(case), _lens(case), case["batch"]
    w, router = _weights(d, seed)
    steps = case.get("steps", 0)
    torch.cuda.synchronize()  # the weights are there before the model's stream reads them
    ctx = P.FirstContext(d, w, router, max_batch=B, max_seq_len=max(lens) + max(steps, 1) + 1, stream=_stream())
    s = SimpleNamespace(case=case, d=d, lens=lens, ctx=ctx, ids=_tokens(d, sum(lens), seed), steps=steps)
    L, D, V = d.n_layers, d.d_model, d.vocab
    s.rho = torch.zeros((B, L), device=DEV)
    if kind == "soft":
        s.targets = _tokens(d, sum(lens), seed + 1)
        s.terms = torch.zeros((B, 4), device=DEV)
        s.hidden = torch.zeros((sum(lens), D), device=DEV)
        torch.cuda.synchronize()
        return s
    s.hidden, s.logits, s.token = torch.zeros((B, D), device=DEV), torch.zeros((B, V), device=DEV), torch.zeros(B, dtype=torch.int32, device=DEV)
    if kind == "generate":
        s.masks, s.last_logits = _masks(case), torch.zeros((B, V), device=DEV)
    if kind == "decode":
        s.masks = _masks(case)
        s.fed = list(_tokens(d, steps * B, seed + 2).view(steps, B).unbind(0))
        s.step_logits = torch.zeros((steps, B, V), device=DEV)
        s.out = list(s.step_logits.unbind(0))
        s.u = torch.rand((B,), generator=torch.Generator(device=DEV).manual_seed(7000 + seed), device=DEV)
    torch.cuda.synchronize()
    if kind == "decode":  # the prompt is there before the steps that are measured
        ctx.prefill_route(s.ids, lens)
        for b, m in enumerate(s.masks):
            ctx.set_mask(b, m)
    return s


# ------------------------------------------------------------------------------------------------ one pass
def _decode(s):
    for fed, out in zip(s.fed, s.out):
        if "top_k" in s.case:
            s.ctx.decode_step_sampled(fed, s.u, 0.8, s.case["top_k"], out, s.token)
        else:
            s.ctx.decode_step(fed, out, s.token)


def run(s):
    kind = s.case["kind"]
    if kind == "lora":  # the adapter goes in, with the next pass out again
        scale = s.sign * 32.0 / s.case["rank"]
        for w, a, b in s.mats.values():
            P.lora_merge(w, a, b, scale)
        s.sign = -s.sign
        return {k: v[0] for k, v in s.mats.items()}
    if kind == "sample":
        P.sample_top_k_static(s.logits, s.u, 0.8, s.case["top_k"], s.token, s.cand)
        return [s.token, s.cand]
    if kind == "soft":
        s.ctx.soft_forward(s.ids, s.lens, s.targets, 0.01, 0.1, s.terms, s.rho, s.hidden)
        return {"terms": s.terms, "rho": s.rho, "hidden": s.hidden}
    if kind == "decode":
        for b, n in enumerate(s.lens):
            s.ctx.set_seq_len(b, n)  # back to the end of the prompt
        _decode(s)
        return {"step_logits": s.step_logits}
    s.ctx.prefill_route(s.ids, s.lens, rho=s.rho, hidden=s.hidden, logits=s.logits, token=s.token)
    out = {"rho": s.rho, "hidden": s.hidden, "logits": s.logits}
    if kind == "generate":
        for b, m in enumerate(s.masks):
            s.ctx.set_mask(b, m)
        for _ in range(s.steps):  # each token goes back in; the logits of the last step are what is looked at
            s.ctx.decode_step(s.token, s.last_logits, s.token)
        out["last_logits"] = s.last_logits
    return out


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "lora":
        e = 2 if case["dtype"] == "bf16" else 4
        r, shapes = case["rank"], _lora_shapes(case).values()
        return {"bytes": sum(2 * e * n * k + 4 * r * (n + k) for n, k in shapes), "flops": sum(2 * r * n * k for n, k in shapes)}
    if kind == "sample":
        return {"bytes": 4 * case["batch"] * (case["vocab"] + case["top_k"] + 2), "flops": 0}
    d, lens = _desc(case), _lens(case)
    e = 2 if d.dtype == "bf16" else 4
    D, nq, nkv, L, V, B = d.d_model, d.n_q_heads * d.head_dim, d.n_kv_heads * d.head_dim, d.n_layers, d.vocab, case["batch"]
    per_layer = D * (2 * nq + 2 * nkv + 3 * d.d_ffn)
    nbytes = flops = 0
    if kind != "decode":  # a prompt pass: all layers on all rows
        rows = sum(lens)
        heads = rows if kind == "soft" else B
        nbytes += e * (per_layer * L + V * D + rows * D) + 4 * (2 * L * D + L * D + D) + 4 * rows
        if kind != "soft":
            nbytes += e * rows * 2 * nkv * L + 4 * B * (V + D + L)
        else:
            nbytes += 4 * rows * D
        flops += 2 * per_layer * L * rows + 2 * V * D * heads + L * sum(2 * nq * n * (n + 1) for n in lens)
    if case.get("steps"):
        masks = _masks(case)
        for t in range(case["steps"]):
            kept = [i for i in range(L) if any(m[i] for m in masks)]
            nbytes += e * (per_layer * len(kept) + V * D + B * D) + 4 * (2 * D * len(kept) + D) + 4 * B * V
            flops += 2 * V * D * B
            for m, n in zip(masks, lens):
                nbytes += e * 2 * nkv * (n + t + 1) * sum(m)
                flops += sum(m) * (2 * per_layer + 4 * nq * (n + t + 1))
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "sample":
        return "exact"
    if kind == "lora":  # one rounding to the storage type, which may fall to the other side of a boundary
        return {"rel": 2e-4, "max": 0.02} if case["dtype"] == "bf16" else {"rel": 5e-7}
    if MODELS[case["model"]][7] == "fp32":
        return {"rel": 2e-5}
    # fp32 sums, activations with 16 significant bits in the prompt pass, K and V rounded to bf16 on the way
    return {"rel": 6e-3}


# ------------------------------------------------------------------------------------------------ the same in 64 bits
def _norm64(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope64(x, pos, base):
    half = x.shape[-1] // 2
    theta = torch.tensor([base ** (-2.0 * i / x.shape[-1]) for i in range(half)], dtype=torch.float64, device=x.device)
    a = pos.double()[:, None] * theta[None, :]
    c, s = torch.cos(a)[:, None, :], torch.sin(a)[:, None, :]
    return torch.cat([x[..., :half] * c - x[..., half:] * s, x[..., half:] * c + x[..., :half] * s], -1)


def _attend64(q, K, V, pos):
    """Rows q [n, Hq, hd] at positions pos over the keys 0 .. pos of K, V [m, Hkv, hd]."""
    n, hq, hd = q.shape
    G, out = hq // K.shape[1], torch.empty_like(q)
    chunk = max(1, (1 << 27) // K.shape[0])
    for r in range(0, n, chunk):
        p = pos[r:r + chunk]
        m = int(p.max()) + 1
        hide = torch.arange(m, device=q.device)[None, :] > p[:, None]
        for h in range(hq):
            sc = q[r:r + chunk, h] @ K[:m, h // G].t().contiguous() / math.sqrt(hd)
            out[r:r + chunk, h] = torch.softmax(sc.masked_fill_(hide, -math.inf), -1) @ V[:m, h // G]
    return out.reshape(n, hq * hd)


def _layer64(d, w, H, pos, past):
    """(phi(H), (K, V) with these rows behind `past`) for rows H at positions pos; K and V as the cache stores them."""
    kvt = torch.bfloat16 if d.dtype == "bf16" else torch.float32
    n = H.shape[0]
    x = _norm64(H, w["attn_norm"], d.rms_eps)
    q = _rope64((x @ w["wq"].t()).view(n, d.n_q_heads, d.head_dim), pos, d.rope_base)
    K = _rope64((x @ w["wk"].t()).view(n, d.n_kv_heads, d.head_dim), pos, d.rope_base).to(kvt).double()
    V = (x @ w["wv"].t()).view(n, d.n_kv_heads, d.head_dim).to(kvt).double()
    if past is not None:
        K, V = torch.cat([past[0], K]), torch.cat([past[1], V])
    att = _attend64(q, K, V, pos) @ w["wo"].t()
    y = _norm64(H + att, w["mlp_norm"], d.rms_eps)
    g = y @ w["w_gate"].t()
    mlp = (g * torch.sigmoid(g) * (y @ w["w_up"].t())) @ w["w_down"].t()
    return att + mlp, (K, V)


def _exact_flops(case):
    """Operations of exact(): the attention there does not leave out the keys behind the diagonal."""
    d, lens = _desc(case), _lens(case)
    return sum(2 * (work(dict(case, kind="prefill", batch=1, lo=n, hi=n, steps=0))["flops"])
               + 2 * d.n_layers * d.n_q_heads * d.head_dim * n * n for n in set(lens)) * len(lens) / len(set(lens))


def exact(case, seed):
    kind = case["kind"]
    if kind == "lora":
        scale = 32.0 / case["rank"]
        return {k: w.double() + scale * (b.double() @ a.double()) for k, (w, a, b) in _lora_inputs(case, seed).items()}
    if kind == "sample":
        return None  # whole numbers
    if _exact_flops(case) > 4e14:
        return None
    d, lens, B, L, steps = _desc(case), _lens(case), case["batch"], _desc(case).n_layers, case.get("steps", 0)
    w, router = _weights(d, seed)
    E = w["embed"]
    prompts = list(_tokens(d, sum(lens), seed).long().split(lens))
    H = [E[p].double() for p in prompts]
    R = [E[t.long()].double() for t in _tokens(d, steps * B, seed + 2).view(steps, B).t().contiguous()] if kind == "decode" else None
    masks = _masks(case) if steps else None
    past = [[None] * L for _ in range(B)]
    rho = torch.zeros((B, L), dtype=torch.float64, device=DEV)
    for i in range(L):
        lw = {k: v.double() for k, v in w["layers"][i].items()}
        for b, n in enumerate(lens):
            score = torch.sigmoid(H[b] @ router[i].double()).mean()
            rho[b, i] = score
            phi, kv = _layer64(d, lw, H[b], torch.arange(n, device=DEV), None)
            if kind == "generate":
                past[b][i] = kv
            if kind == "decode" and masks[b][i]:
                R[b] = R[b] + _layer64(d, lw, R[b], torch.arange(n, n + steps, device=DEV), kv)[0]
            H[b] = H[b] + (score * phi if kind == "soft" else phi)
            del phi, kv
        del lw

    def head(x):
        y = _norm64(x, w["final_norm"], d.rms_eps)
        return torch.cat([y @ part.double().t() for part in w["lm_head"].split(16384)], -1)

    if kind == "soft":
        terms, targets = torch.zeros((B, 4), dtype=torch.float64, device=DEV), _tokens(d, sum(lens), seed + 1).long().split(lens)
        for b in range(B):
            ce = torch.nn.functional.cross_entropy(head(H[b]), targets[b])
            reg, pp = router.double().square().sum(), rho[b].sum()
            terms[b] = torch.stack([ce, reg, pp, ce + 0.01 * reg + 0.1 * pp])
        return {"terms": terms, "rho": rho, "hidden": torch.cat(H)}
    if kind == "decode":
        return {"step_logits": torch.stack([head(r) for r in R], 1)}
    last = torch.stack([h[-1] for h in H])
    out = {"rho": rho, "hidden": last, "logits": head(last)}
    if kind == "generate":
        logits = out["logits"]
        for t in range(steps):
            rows = E[logits.argmax(-1)].double()
            for b, n in enumerate(lens):
                for i in range(L):
                    if masks[b][i]:
                        lw = {k: v.double() for k, v in w["layers"][i].items()}
                        phi, past[b][i] = _layer64(d, lw, rows[b:b + 1], torch.full((1,), n + t, device=DEV), past[b][i])
                        rows[b] += phi[0]
            logits = head(rows)
        out["last_logits"] = logits
    return out
