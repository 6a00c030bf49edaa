"""The work that a program built on this library has it do, as cases that can be timed and compared.

A case is a dict of plain values.  Three kinds:
  loop    one generation call on a three-model stack (prompt ingestion, draft / verify / accept loop, roll back): the
          three-model loop, the two-model baseline or plain sampling; then the logits of the prompt's last tokens
  ingest  a prompt goes into one model's KV cache, then the logits of its last token (what precedes the first sample)
  accept  the acceptance stage on logits that are on the device already: one stage as a serving loop calls it, or many
          stages per call as an evaluation does
Sizes are those of the package's stack configurations (tiny, small, paper = 1B / 3B / 8B shapes, long) and, for the
draws, other depths, prompt lengths, widths, windows, vocabularies and thresholds of the same ranges.  Single layers are
what a change of a kernel shows best, so the big shapes are mostly taken with fewer layers; one case has all of them.
Weights are N(0, 0.02^2) as everywhere in this repository, norm gains are 1, prompts are uniform token ids.
"""
import math

import numpy as np
import torch

import paper_2510_12966_amd as psd

# d_model, heads, kv heads, d_ffn
SHAPES = {
    "tiny_draft": (64, 4, 2, 256), "tiny_qualifier": (128, 4, 2, 512), "tiny_target": (256, 8, 4, 1024),
    "small_draft": (512, 8, 4, 1408), "small_qualifier": (1024, 16, 4, 2816), "small_target": (2048, 16, 8, 5632),
    "paper_draft": (2048, 32, 8, 8192), "paper_qualifier": (3072, 24, 8, 8192), "paper_target": (4096, 32, 8, 14336),
    "stub": (64, 2, 1, 64),   # the two models of a context that a single-model case does not use
}
ROLES = ("draft", "qualifier", "target")
DEPTH = {"tiny": (2, 4, 6), "small": (4, 8, 12), "paper": (16, 28, 32)}
THETA = {"tiny": 10000.0, "small": 10000.0, "paper": 500000.0}
EPS = 1e-5
TAIL = 4   # prompt tokens whose logits a loop case returns


def listed():
    return [
        # the tiny fp32 stack, whole loop: the smallest models, where launches and latency are everything
        dict(name="loop_tiny_fp32", kind="loop", mode="psd", family="tiny", dtype="f32", ld=2, lq=4, lt=6, vocab=512, prompt=16, new=64,
             k1=4, k2=8, tq=0.004, tt=0.012),
        # the small bf16 stack, thresholds inside its divergence range: rejections, replacement draws, rollbacks
        dict(name="loop_small", kind="loop", mode="psd", family="small", dtype="bf16", ld=4, lq=8, lt=12, vocab=32000, prompt=128, new=64,
             k1=4, k2=8, tq=0.0722, tt=0.135),
        # the headline workload: 1B / 3B / 8B shapes at full depth, window 10
        dict(name="loop_paper", kind="loop", mode="psd", family="paper", dtype="bf16", ld=16, lq=28, lt=32, vocab=128256, prompt=512, new=176,
             k1=5, k2=10, tq=0.5, tt=0.3),
        # long context and a long window: attention over thousands of keys, 17-token verify passes (a quarter of the layers)
        dict(name="loop_long", kind="loop", mode="psd", family="paper", dtype="bf16", ld=4, lq=7, lt=8, vocab=128256, prompt=4001, new=136,
             k1=8, k2=16, tq=0.5, tt=0.3),
        # the widest windows the interface takes: verify passes of 13 and 31 tokens
        dict(name="loop_wide", kind="loop", mode="psd", family="paper", dtype="bf16", ld=2, lq=4, lt=4, vocab=128256, prompt=131, new=124,
             k1=12, k2=30, tq=0.5, tt=0.3),
        # the two-model baseline, exact speculative sampling: most proposals are refused
        dict(name="sd_strict", kind="loop", mode="sd", family="paper", dtype="bf16", ld=4, lq=1, lt=8, vocab=128256, prompt=77, new=16,
             k1=4, k2=4, tq=0.0, tt=0.0),
        # plain sampling from the target: one token a pass
        dict(name="plain_target", kind="loop", mode="plain", family="paper", dtype="bf16", ld=1, lq=1, lt=8, vocab=128256, prompt=33, new=16,
             k1=1, k2=1, tq=0.0, tt=0.0),
        # prompt ingestion, the target's shape, a full pass less a few tokens
        dict(name="ingest_target", kind="ingest", shape="paper_target", layers=4, vocab=32000, prompt=509),
        # a long prompt into the draft's shape: several passes, attention over what is cached already
        dict(name="ingest_draft_long", kind="ingest", shape="paper_draft", layers=4, vocab=32000, prompt=3000),
        # a short prompt: less than one column group of the widest passes
        dict(name="ingest_short", kind="ingest", shape="paper_qualifier", layers=4, vocab=32000, prompt=100),
        # one acceptance stage at the headline window, as the loop and a serving program call it
        dict(name="accept_one", kind="accept", trials=1, k=10, vocab=128256, rho=0.8, T=0.2),
        # many stages per call (threshold sweeps over recorded logits)
        dict(name="accept_many", kind="accept", trials=48, k=8, vocab=128256, rho=0.8, T=0.2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("loop", "loop", "loop", "ingest", "ingest", "accept"))
    if kind == "accept":
        trials, k, vocab = _log_int(rng, 1, 48), _log_int(rng, 1, 32), rng.choice((32000, 128256, 50257, 128255))
        return dict(kind="accept", trials=max(1, min(trials, 48 * 8 * 128256 // (k * vocab))), k=k, vocab=vocab, rho=rng.choice((0.5, 0.8, 0.95)),
                    T=round(rng.uniform(0.0, 0.5), 3))
    if kind == "ingest":
        role = rng.choice(ROLES)
        return dict(kind="ingest", shape="%s_%s" % (rng.choice(("small", "paper", "paper")), role), layers=rng.randint(1, 4), vocab=rng.choice((32000, 32003, 128256)),
                    prompt=_log_int(rng, 20, 3000 if role == "draft" else 1200))
    family = rng.choice(("tiny", "small", "paper", "paper"))
    mode = rng.choice(("psd", "psd", "sd", "plain"))
    deep = DEPTH[family] if family != "paper" else (4, 4, 4)
    ld, lq, lt = (rng.randint(1, n) for n in deep)
    k2 = rng.randint(1, 31) if mode == "psd" else rng.randint(1, 12)
    k1 = rng.randint(1, min(30, k2)) if mode == "psd" else k2
    tq, tt = rng.choice(((0.7, 0.7), (0.5, 0.3), (0.0, 0.0))) if mode != "plain" else (0.0, 0.0)
    new = rng.randint(8, 16) if tt == 0.0 else rng.randint(16, 48)
    vocab = rng.choice((512, 1001)) if family == "tiny" else rng.choice((32000, 32003)) if family == "small" else rng.choice((32000, 32003, 128256))
    return dict(kind="loop", mode=mode, family=family, dtype="f32" if family == "tiny" else "bf16", ld=ld, lq=lq, lt=lt, vocab=vocab,
                prompt=_log_int(rng, 5, 64 if family == "tiny" else 2000), new=new, k1=k1, k2=k2, tq=tq, tt=tt)


# ---- weights ---------------------------------------------------------------------------------------------------------
def _sizes(shape, layers, vocab):
    """Elements of the blob's tensors in order: [(is_norm, elements)], and which belong to a layer."""
    d, H, KV, F = SHAPES[shape]
    kv = KV * (d // H)
    layer = [(True, d), (False, (d + 2 * kv) * d), (False, d * d), (True, d), (False, 2 * F * d), (False, d * F)]
    return [(False, vocab * d)] + layer * layers + [(True, d)]


def _tensors(shape, layers, vocab, seed, dtype):
    """The blob's tensors one after the other, on the GPU."""
    for i, (norm, n) in enumerate(_sizes(shape, layers, vocab)):
        if norm:
            yield torch.ones(n, dtype=dtype, device="cuda")
        else:
            g = torch.Generator(device="cuda").manual_seed(seed * 1000 + i)
            yield torch.empty(n, dtype=dtype, device="cuda").normal_(0.0, 0.02, generator=g)


def _desc(shape, layers, vocab, theta, seed, f32=False):
    dtype = torch.float32 if f32 else torch.bfloat16
    total = sum(n for _, n in _sizes(shape, layers, vocab))
    host = torch.empty(total, dtype=dtype, pin_memory=True)
    at = 0
    for t in _tensors(shape, layers, vocab, seed, dtype):
        host[at:at + t.numel()].copy_(t)
        at += t.numel()
    blob = host.numpy() if f32 else host.view(torch.int16).numpy().view(np.uint16)
    d, H, KV, F = SHAPES[shape]
    return psd.ModelDesc(layers, d, H, KV, F, vocab, theta, psd.F32 if f32 else psd.BF16, blob, EPS)


def _prompt(seed, n, vocab):
    return np.random.default_rng([seed, 77]).integers(0, vocab, n).astype(np.int32)


def _models(case):
    """(shape, layers) per role, and the rotary base."""
    if case["kind"] == "loop":
        return [("%s_%s" % (case["family"], r), case[l]) for r, l in zip(ROLES, ("ld", "lq", "lt"))], THETA[case["family"]]
    return [("stub", 1), ("stub", 1), (case["shape"], case["layers"])], THETA["paper"]


def _seed_of(seed, role):
    return (seed * 3 + role) % (1 << 40)


def prepare(case, seed):
    if case["kind"] == "accept":
        B, k, V = case["trials"], case["k"], case["vocab"]
        g = torch.Generator(device="cuda").manual_seed(seed)
        p = torch.empty(B, k + 1, V, device="cuda").normal_(0.0, 3.0, generator=g)
        q = torch.empty(B, k, V, device="cuda").normal_(0.0, 3.0, generator=g)
        q.mul_(math.sqrt(1.0 - case["rho"] ** 2)).add_(p[:, :k], alpha=case["rho"])
        tokens = torch.empty(B, k, dtype=torch.int32, device="cuda")
        for b in range(B):   # proposals are samples of their rows
            u = torch.rand(k, V, device="cuda", generator=g).clamp_min_(1e-20)
            tokens[b] = (q[b] - torch.log(-torch.log(u))).argmax(-1)
        out = dict(n=torch.empty(B, dtype=torch.int32, device="cuda"), tok=torch.empty(B, dtype=torch.int32, device="cuda"),
                   div=torch.empty(B, k, device="cuda"))
        ws = torch.empty(psd.accept_workspace_bytes(B, k, V), dtype=torch.uint8, device="cuda")
        psd.accept_noalloc_init()
        return dict(case=case, p=p, q=q, tokens=tokens, out=out, ws=ws, seed=seed & 0xffffffff)
    models, theta = _models(case)
    f32 = case.get("dtype") == "f32"
    descs = [_desc(s, n, case["vocab"], theta, _seed_of(seed, i), f32) for i, (s, n) in enumerate(models)]
    k1, k2 = case.get("k1", 1), case.get("k2", 1)
    max_seq = case["prompt"] + case.get("new", 0) + k2 + 8
    ctx = psd.Context(*descs, case.get("tq", 0.0), case.get("tt", 0.0), k1, k2, max_seq, flags=psd.FLAG_GRAPH)
    return dict(case=case, ctx=ctx, prompt=_prompt(seed, case["prompt"], case["vocab"]), seed=seed & 0xffffffff)


def run(state):
    case = state["case"]
    if case["kind"] == "accept":
        o, B, k, V = state["out"], case["trials"], case["k"], case["vocab"]
        args = (state["p"], state["q"], state["tokens"], B, k, V, case["T"], 1.0, state["seed"], 100, 2, True, o["n"], o["tok"], o["div"])
        if B == 1:
            psd.accept_batch_noalloc(*args)
        else:
            psd.accept_batch(*args, state["ws"], state["ws"].numel())
        return dict(o)
    ctx, prompt = state["ctx"], state["prompt"]
    n = prompt.size
    if case["kind"] == "ingest":
        at = 0
        while at < n - 1:
            w = min(512 if SHAPES[case["shape"]][0] >= 512 else 128, n - 1 - at)
            ctx.forward(2, prompt[at:at + w], at, want_logits=False)
            at += w
        return dict(logits=ctx.forward(2, prompt[n - 1:], n - 1))
    if case["mode"] == "psd":
        tokens, _ = ctx.generate(prompt, case["new"], state["seed"])
    elif case["mode"] == "sd":
        tokens, _ = ctx.generate_sd(0, case["k2"], case["tt"], prompt, case["new"], state["seed"])
    else:
        tokens, _ = ctx.generate_plain(2, prompt, case["new"], state["seed"])
    t = min(TAIL, n)
    return dict(tokens=tokens, logits=ctx.forward(2, prompt[n - t:], n - t))


# ---- what a pass cannot do without ------------------------------------------------------------------------------------
def _passes(case):
    """Fewest passes of each model: every proposal accepted.  [(tokens, logit rows)] per role, in order, after the prompt."""
    d, q, t = [], [], []
    done = 0
    while done < case["new"]:
        if case["mode"] == "plain":
            t.append((1, 1))
            done += 1
            continue
        k2 = case["k2"]
        if case["mode"] == "sd":
            d += [(1, 1)] * k2
        else:
            filled = 0
            while filled < k2:
                m = min(case["k1"], k2 - filled)
                d += [(1, 1)] * m
                q.append((m + 1, m + 1))
                filled += m + (filled + m < k2)
        t.append((k2 + 1, k2 + 1))
        done += k2 + 1
    return d, q, t


def _model_work(shape, layers, vocab, el, prompt, passes):
    """bytes and flops of one model: the prompt in passes of 512, then the given passes."""
    d, H, KV, F = SHAPES[shape]
    kv = KV * (d // H)
    per_layer = (2 * d + 2 * kv) * d + 3 * d * F
    nb = nf = 0.0
    ctx = 0
    todo = [(min(512, prompt - a), 0) for a in range(0, prompt, 512)] + list(passes)
    for w, rows in todo:
        ctx += w
        nb += layers * (per_layer * el + 2 * kv * el * ctx) + (vocab * d * el + rows * vocab * 4 if rows else 0)
        nf += 2.0 * w * layers * (per_layer + 2 * d * (ctx - w / 2)) + 2.0 * rows * vocab * d
    return nb, nf


def work(case):
    if case["kind"] == "accept":
        n = case["trials"] * (2 * case["k"] + 1) * case["vocab"]
        return {"bytes": 4.0 * n, "flops": 10.0 * n}
    el = 4 if case.get("dtype") == "f32" else 2
    if case["kind"] == "ingest":
        nb, nf = _model_work(case["shape"], case["layers"], case["vocab"], el, case["prompt"] - 1, [(1, 1)])
        return {"bytes": nb, "flops": nf}
    models, _ = _models(case)
    per_role = list(_passes(case))
    per_role[2] = per_role[2] + [(min(TAIL, case["prompt"]),) * 2]
    used = {"psd": (0, 1, 2), "sd": (0, 2), "plain": (2,)}[case["mode"]]
    nb = nf = 0.0
    for r in used:
        b, f = _model_work(models[r][0], models[r][1], case["vocab"], el, case["prompt"] - 1, per_role[r])
        nb, nf = nb + b, nf + f
    return {"bytes": nb, "flops": nf}


def tolerance(case):
    if case["kind"] == "accept":
        return {"rel": 2e-6, "max": 8e-6, "differ": 0.01}   # divergences are 32-bit sums over the vocabulary
    if case.get("dtype") == "f32":
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.01}
    # bf16 weights, activations and KV as bf16 pairs (2^-17), 32-bit sums; differences grow through the layers
    return {"rel": 2e-4, "max": 2e-3, "differ": 0.01}


# ---- the same in 64 bits -------------------------------------------------------------------------------------------------
def _logits64(shape, layers, vocab, theta, seed, f32, tokens, rows):
    """Logits of the last `rows` tokens, plain torch in float64, one layer's weights at a time."""
    d, H, KV, F = SHAPES[shape]
    hd, n = d // H, len(tokens)
    kv = KV * hd
    it = _tensors(shape, layers, vocab, seed, torch.float32 if f32 else torch.bfloat16)
    f64 = lambda t, *s: t.double().view(*s)  # noqa: E731
    embed = next(it)
    x = embed.view(vocab, d)[torch.as_tensor(tokens, dtype=torch.int64, device="cuda")].double()
    pos = torch.arange(n, device="cuda", dtype=torch.float64)
    ang = pos[:, None] * theta ** (-2.0 * torch.arange(hd // 2, device="cuda", dtype=torch.float64) / hd)
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]
    norm = lambda v, g: v * torch.rsqrt(v.square().mean(-1, keepdim=True) + EPS) * g.double()  # noqa: E731

    def rotate(v):
        a, b = v[..., :hd // 2], v[..., hd // 2:]
        return torch.cat((a * cos - b * sin, b * cos + a * sin), -1)

    hidden = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
    for _ in range(layers):
        h = norm(x, next(it))
        qkv = h @ f64(next(it), d + 2 * kv, d).t()
        q, k, v = qkv[:, :d].reshape(n, H, hd), qkv[:, d:d + kv].reshape(n, KV, hd), qkv[:, d + kv:].reshape(n, KV, hd)
        q, k = rotate(q), rotate(k)
        out = torch.empty(n, H, hd, dtype=torch.float64, device="cuda")
        for j in range(H):
            s = (q[:, j] @ k[:, j * KV // H].t()) / math.sqrt(hd)
            out[:, j] = s.masked_fill_(hidden, -math.inf).softmax(-1) @ v[:, j * KV // H]
        x = x + out.reshape(n, d) @ f64(next(it), d, d).t()
        h = norm(x, next(it))
        gu = h @ f64(next(it), 2 * F, d).t()
        x = x + (torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]) @ f64(next(it), d, F).t()
    h = norm(x[n - rows:], next(it))
    return (h @ f64(embed, vocab, d).t()).cpu()


def exact(case, seed):
    if case["kind"] == "accept":
        s = prepare(case, seed)
        div = torch.empty(case["trials"], case["k"], dtype=torch.float64)
        for b in range(case["trials"]):
            lp, lq = s["p"][b, :case["k"]].double().log_softmax(-1), s["q"][b].double().log_softmax(-1)
            lm = torch.logaddexp(lp, lq) - math.log(2.0)
            div[b] = 0.5 * ((lp.exp() * (lp - lm)).sum(-1) + (lq.exp() * (lq - lm)).sum(-1)).cpu()
        return dict(n=None, tok=None, div=div)
    models, theta = _models(case)
    shape, layers = models[2]
    rows = 1 if case["kind"] == "ingest" else min(TAIL, case["prompt"])
    lg = _logits64(shape, layers, case["vocab"], theta, _seed_of(seed, 2), case.get("dtype") == "f32", _prompt(seed, case["prompt"], case["vocab"]), rows)
    return dict(logits=lg) if case["kind"] == "ingest" else dict(tokens=None, logits=lg)
