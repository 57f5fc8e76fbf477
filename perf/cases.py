"""Performance cases of the loss stage: what a training or scoring program calls, at the sizes
it calls it with, through the package's public entry points.

Kinds of case (the "kind" entry) and what they stand for:
  step       one training step's loss stage: the fused call on materialised logits (log-prob,
             ratios, decisions, loss, dlogits), then the PPO-EWMA step of the per-token proxy
             with its reset rule on the device
  loss       the fused call alone, as a training loop with exact old log-probs makes it
  autograd   the same stage inside a model's autograd graph (DecoupledPPOLoss), a fraction of
             the positions masked (tool output), the loss scaled for gradient accumulation
  logprob    sampled-token log-probs of a scoring pass; with versions > 1, of a partial-rollout
             batch whose tokens come from several policy versions
  shard      one GPU's share of a vocabulary-parallel loss stage
  ewma       the PPO-EWMA update of a parameter shard
  lm_head    the loss stage with the LM head folded in, both gradients: the plain call
             ("call"), inside autograd ("autograd"), or on the library's own scratch
             ("noalloc")
"""
from __future__ import annotations

import math

import torch

import paper_2605_12070_amd as P

DEV = "cuda"
BAND = (0.5, 2.0)
EPS = (0.2, 0.2)
SEQ = 512
WINDOW = 6                    # versions a rollout may span: the proxy's decay is 6 / 8
# No token's ratio lies closer than this (in log) to a band or clip bound: a decision on the
# bound itself would turn on the last bit of a log-prob.
MARGIN = 2e-3
LARGEST = 16384 * 151936      # entries of the largest bf16 logits matrix
LM_LARGEST = 8192 * 4096 * 151936


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest training step: one short fp32 batch, where launches and host work count
        dict(name="step_tiny_f32", kind="step", dtype="f32", T=256, V=1024, mask=0.0),
        # a 32000-entry vocabulary, 16 sequences of 256 tokens
        dict(name="step_small_vocab", kind="step", dtype="bf16", T=4096, V=32000, mask=0.0),
        # the benchmark's own step: 32 sequences of 512 tokens over a 151936-entry vocabulary
        dict(name="step_large_vocab", kind="step", dtype="bf16", T=16384, V=151936, mask=0.0),
        # an agentic batch in a model's graph: 40 % of the positions are tool output
        dict(name="autograd_agentic", kind="autograd", dtype="bf16", T=8192, V=151936, mask=0.4),
        # a trainer that upcasts its logits: fp32 rows of an odd vocabulary, contiguous, so the
        # rows start anywhere
        dict(name="loss_f32_odd_vocab", kind="loss", dtype="f32", T=4096, V=50257, mask=0.0,
             ref="given", grads=True),
        # old log-probs of a scoring pass over an odd vocabulary
        dict(name="logprob_odd_vocab", kind="logprob", dtype="bf16", T=8192, V=151937, versions=1),
        # exact old log-probs of a partial-rollout batch, four policy versions
        dict(name="logprob_versions", kind="logprob", dtype="bf16", T=4096, V=151936, versions=4),
        # one of eight vocabulary shards of the large step
        dict(name="shard_step", kind="shard", dtype="bf16", T=16384, V=151936, P=8),
        # the proxy of a quarter-billion-parameter shard, fp32 master weights
        dict(name="ewma_params", kind="ewma", dtype="f32", n=1 << 28),
        # the folded LM head at full size
        dict(name="lm_head_full", kind="lm_head", api="call", T=8192, d=4096, V=151936, mask=0.0),
        # a micro-batch through autograd
        dict(name="lm_head_micro", kind="lm_head", api="autograd", T=1024, d=2048, V=32000, mask=0.0),
        # a loop that may not allocate: the library's 64 MiB scratch, vocabulary in chunks
        dict(name="lm_head_noalloc", kind="lm_head", api="noalloc", T=2048, d=4096, V=151936, mask=0.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "loss", "loss", "autograd", "logprob", "logprob", "shard", "ewma",
                       "lm_head", "lm_head", "lm_head"])
    if kind == "ewma":
        return dict(kind=kind, dtype=rng.choice(["f32", "bf16"]), n=_log_int(rng, 1 << 14, 1 << 28))
    if kind == "lm_head":
        api = rng.choice(["call", "autograd", "noalloc"])
        T = _log_int(rng, 128, 4096 if api == "noalloc" else 8192)
        d = 8 * _log_int(rng, 64, 512)
        V = _log_int(rng, 2000, 151936)
        V = V if rng.random() < 0.5 else 8 * (V // 8)
        # the no-allocation form forms the logits twice
        most = LM_LARGEST // (2 if api == "noalloc" else 1)
        T = max(1, min(T, most // (d * V)))
        return dict(kind=kind, api=api, T=T, d=d, V=V, mask=rng.choice([0.0, 0.3]))
    dtype = rng.choice(["bf16", "bf16", "f32"])
    es = 4 if dtype == "f32" else 2
    V = _log_int(rng, 1000, 262144)
    if rng.random() < 0.5:
        V = 16 * (V // 16)
    T = _log_int(rng, 128, 16384)
    # passes over the logits' bytes against the largest step's read and write
    passes = {"step": 2, "loss": 2, "autograd": 4, "logprob": 1, "shard": 3}[kind]
    T = max(1, min(T, 2 * LARGEST * 2 // (passes * V * es)))
    if kind == "logprob":
        versions = rng.choice([1, 1, 2, 4])
        T = max(1, min(T, 2 * LARGEST // (versions * V * es)))
        return dict(kind=kind, dtype=dtype, T=T, V=V, versions=versions)
    if kind == "shard":
        # shards are cut on multiples of 16 columns (padded vocabularies)
        shards = rng.choice([2, 4, 8])
        return dict(kind=kind, dtype=dtype, T=T, V=16 * shards * max(1, V // (16 * shards)), P=shards)
    c = dict(kind=kind, dtype=dtype, T=T, V=V, mask=rng.choice([0.0, 0.4]))
    if kind == "loss":
        c["ref"] = rng.choice(["given", "given", "log_linear"])
        c["grads"] = rng.random() < 0.75
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _rows(T, V):
    """Rows of a [rows, V] float32 slice of at most 1 GiB."""
    return max(1, min(T, (1 << 28) // V))


def _logits(T, V, dtype, gen):
    """N(0, 3^2) logits, 1 % of the rows with one entry 15 higher (a confident token)."""
    z = torch.empty(T, V, dtype=dtype, device=DEV)
    n = _rows(T, V)
    for a in range(0, T, n):
        b = min(T, a + n)
        z[a:b] = (3.0 * torch.randn(b - a, V, generator=gen, device=DEV)).to(dtype)
    k = max(1, T // 100)
    rows = torch.randperm(T, generator=gen, device=DEV)[:k]
    cols = torch.randint(0, V, (k,), generator=gen, device=DEV)
    z[rows, cols] += 15.0
    return z


def _sample(z, gen):
    """Token ids drawn from softmax(z) and their log-probs (float32 rows in slices)."""
    T, V = z.shape
    ids = torch.empty(T, dtype=torch.int64, device=DEV)
    lp = torch.empty(T, dtype=torch.float64, device=DEV)
    n = _rows(T, V)
    for a in range(0, T, n):
        b = min(T, a + n)
        x = z[a:b].float()
        q = torch.empty_like(x).exponential_(generator=gen).log_()
        ids[a:b] = torch.argmax(x - q, dim=1)
        lp[a:b] = (x.gather(1, ids[a:b, None])[:, 0] - torch.logsumexp(x, dim=1)).double()
    return ids, lp


def _away(x, bounds):
    """x with the values near a bound moved off it."""
    for b in bounds:
        x = torch.where((x - b).abs() < MARGIN, b + 2 * MARGIN, x)
    return x


def _tokens(T, anchor, gen, mask, ref="given"):
    """Reference and behaviour log-probs (staleness drift, train-inference discrepancy with
    a few large jumps), per-sequence advantages and the loss mask (spans of tool output)."""
    log_r_s = _away(0.2 * torch.randn(T, generator=gen, device=DEV, dtype=torch.float64),
                    [math.log(1 - EPS[0]), math.log(1 + EPS[1])])
    u = torch.rand(2, T, generator=gen, device=DEV, dtype=torch.float64)
    lap = 0.05 * (torch.log1p(-u[0]) - torch.log1p(-u[1]))
    jump = (torch.rand(T, generator=gen, device=DEV) < 0.05) * \
        (2.0 * torch.randint(0, 2, (T,), generator=gen, device=DEV) - 1.0)
    log_r_d = _away(lap + jump, [math.log(BAND[0]), math.log(BAND[1])])
    lp_ref = (anchor - log_r_s).float()
    lp_mu = (lp_ref.double() - log_r_d).float()
    if ref == "log_linear":       # both ratios are powers of pi_theta / mu_old
        total = _away(log_r_s + log_r_d, [2 * math.log(b) for b in
                                          (1 - EPS[0], 1 + EPS[1], BAND[0], BAND[1])])
        lp_ref, lp_mu = None, (anchor - total).float()
    n_seq = -(-T // SEQ)
    adv = torch.randn(n_seq, generator=gen, device=DEV).repeat_interleave(SEQ)[:T].contiguous()
    m = torch.ones(T, dtype=torch.uint8, device=DEV)
    if mask > 0:                  # alternating spans, mean length 300 kept and 300 p / (1 - p) not
        span = torch.arange(T, device=DEV) % int(300 / (1 - mask))
        shift = int(torch.randint(0, 300, (1,), generator=gen, device=DEV))
        m = (span.roll(shift) < 300).to(torch.uint8) if T > 600 else \
            (torch.rand(T, generator=gen, device=DEV) >= mask).to(torch.uint8)
    return dict(lp_ref=lp_ref, lp_mu=lp_mu, adv=adv, mask=m)


def _lm_inputs(case, gen):
    T, d, V = case["T"], case["d"], case["V"]
    hidden = torch.randn(T, d, generator=gen, device=DEV).to(torch.bfloat16)
    weight = torch.empty(V, d, dtype=torch.bfloat16, device=DEV)
    std = 1.28 / math.sqrt(d)                  # logit std 1.28 at any width
    for a in range(0, V, 16384):
        b = min(V, a + 16384)
        weight[a:b] = (std * torch.randn(b - a, d, generator=gen, device=DEV)).to(torch.bfloat16)
    ids = torch.empty(T, dtype=torch.int64, device=DEV)
    anchor = torch.empty(T, dtype=torch.float64, device=DEV)
    n = _rows(T, V)
    wf = weight.float()
    for a in range(0, T, n):
        b = min(T, a + n)
        ids[a:b], anchor[a:b] = _sample(hidden[a:b].float() @ wf.T, gen)
    del wf
    return dict(hidden=hidden, weight=weight, ids=ids, **_tokens(T, anchor, gen, case["mask"]))


def _inputs(case, seed):
    """Everything a case's call takes, from the seed alone."""
    gen = _gen(seed)
    kind = case["kind"]
    if kind == "ewma":
        n, dt = case["n"], _dtype(case)
        x0 = (0.02 * torch.randn(n, generator=gen, device=DEV)).to(dt)
        x = torch.randn(n, generator=gen, device=DEV).mul_(1e-3).add_(x0.float()).to(dt)
        stats = torch.tensor([4096, 4000, 3900, 3850, 0], dtype=torch.int32, device=DEV)
        return dict(x0=x0, x=x, stats=stats)
    if kind == "lm_head":
        return _lm_inputs(case, gen)
    T, V = case["T"], case["V"]
    z = _logits(T, V, _dtype(case), gen)
    if kind == "logprob":
        mats = [z] + [_logits(T, V, z.dtype, gen) for _ in range(case["versions"] - 1)]
        ids = torch.randint(0, V, (T,), generator=gen, device=DEV)
        s = dict(mats=mats, ids=ids)
        if case["versions"] > 1:  # segments of a rollout, the stalest first
            cut = torch.randint(64, 512, (1,), generator=gen, device=DEV).item()
            s["ver"] = (torch.arange(T, device=DEV) // cut % case["versions"]).to(torch.int32)
        return s
    ids, anchor = _sample(z, gen)
    s = dict(ids=ids, **_tokens(T, anchor, gen, case.get("mask", 0.0), case.get("ref", "given")))
    if kind == "shard":
        Vs = V // case["P"]
        shards = z.float().view(T, case["P"], Vs) if T * V < (1 << 30) else None
        lse = torch.logsumexp(shards, dim=2) if shards is not None else torch.cat(
            [torch.logsumexp(z[a:a + 2048].float().view(-1, case["P"], Vs), dim=2)
             for a in range(0, T, 2048)])
        zy = z.gather(1, ids[:, None])[:, 0].float()
        mine = ids < Vs                                   # this GPU holds the first columns
        s.update(shard=z[:, :Vs].contiguous(), gathered=lse.T.contiguous(),
                 zy_others=torch.where(mine, torch.zeros_like(zy), zy))
        return s
    s["z"] = z
    if kind == "step":            # the proxy holds the tokens' earlier reference log-probs
        s["x0"] = s["lp_ref"] + 0.1 * torch.randn(T, generator=gen, device=DEV)
    if kind == "loss":
        s["tscale"] = torch.rand(T, generator=gen, device=DEV) + 0.5
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind = case["kind"]
    if kind in ("step", "ewma"):
        # about four tokens in five are active: the reset rule runs and does not fire
        s["proxy"] = P.EwmaProxyDevice(s["x0"], beta=P.beta_from_window(WINDOW), tau=0.6, patience=1)
    if kind == "step":                        # a loop keeps its gradient buffer
        s["dlogits"] = torch.empty_like(s["z"])
    if kind == "autograd":
        s["z"].requires_grad_(True)
    if kind == "lm_head" and case["api"] == "autograd":
        s["hidden"].requires_grad_(True)
        s["weight"].requires_grad_(True)
    if kind == "lm_head" and case["api"] == "call":      # a loop keeps its buffers
        s["out"] = None
    return s


# ------------------------------------------------------------------ one pass
ACCUM = 0.25          # gradient-accumulation factor of the autograd cases


def _fields(r):
    return dict(loss=r.loss, logp=r.logp, loss_tok=r.loss_tok, flags=r.flags, stats=r.stats)


def _proxy(p):
    return dict(x=p.x, w=p.state[:1].view(torch.float64), count=p.state[1:3].view(torch.int32))


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "step":
        r = P.decoupled_ppo_loss_fwd_bwd(s["z"], s["ids"], s["lp_mu"], s["lp_ref"], s["adv"],
                                         s["mask"], band=BAND, clip_eps=EPS, dlogits=s["dlogits"])
        s["proxy"].step(s["lp_ref"], r.stats)
        return dict(_fields(r), dlogits=r.dlogits, proxy=_proxy(s["proxy"]))
    if kind == "loss":
        r = P.decoupled_ppo_loss_fwd_bwd(s["z"], s["ids"], s["lp_mu"], s["lp_ref"], s["adv"],
                                         s["mask"], s["tscale"], band=BAND, clip_eps=EPS,
                                         ref_mode=case["ref"], want_dlogits=case["grads"])
        return dict(_fields(r), dlogits=r.dlogits)
    if kind == "autograd":
        loss, lp, stats = P.DecoupledPPOLoss.apply(s["z"], s["ids"], s["lp_mu"], s["lp_ref"],
                                                   s["adv"], s["mask"], None, None)
        (g,) = torch.autograd.grad(loss * ACCUM, s["z"])
        return dict(loss=loss.detach(), logp=lp, stats=stats, dlogits=g)
    if kind == "logprob":
        if case["versions"] == 1:
            lp, lse = P.logprob_fwd(s["mats"][0], s["ids"], with_lse=True)
        else:
            lp, lse = P.logprob_fwd_versioned(s["mats"], s["ver"], s["ids"], with_lse=True)
        return dict(logp=lp, lse=lse)
    if kind == "shard":
        lse, zy = P.vocab_shard_stats(s["shard"], s["ids"], 0, case["V"], s["mask"])
        s["gathered"][0].copy_(lse)                       # the exchange's local half
        zy = zy + s["zy_others"]
        full = P.vocab_shard_combine(s["gathered"])
        r = P.decoupled_ppo_loss_shard_fwd_bwd(s["shard"], 0, case["V"], full, zy, s["ids"],
                                               s["lp_mu"], s["lp_ref"], s["adv"], s["mask"],
                                               band=BAND, clip_eps=EPS)
        return dict(_fields(r), shard_lse=lse, zy=zy, lse=full, dlogits=r.dlogits)
    if kind == "ewma":
        s["proxy"].step(s["x"], s["stats"])
        return _proxy(s["proxy"])
    args = (s["hidden"], s["weight"], s["ids"], s["lp_mu"], s["lp_ref"], s["adv"], s["mask"])
    if case["api"] == "autograd":
        loss, lp, stats = P.FusedLMHeadLoss.apply(*args, None, None)
        gh, gw = torch.autograd.grad(loss * ACCUM, (s["hidden"], s["weight"]))
        return dict(loss=loss.detach(), logp=lp, stats=stats, dhidden=gh, dweight=gw)
    if case["api"] == "noalloc":
        r, _ = P.fused_lm_head_loss_fwd_bwd_noalloc(*args, band=BAND, clip_eps=EPS)
    else:
        r = s["out"] = P.fused_lm_head_loss_fwd_bwd(*args, band=BAND, clip_eps=EPS, out=s["out"])
    return dict(_fields(r), dhidden=r.dhidden, dweight=r.dweight)


# ------------------------------------------------------------------ what a pass needs
def work(case):
    kind = case["kind"]
    if kind == "ewma":
        es = 4 if case["dtype"] == "f32" else 2
        return dict(bytes=3 * case["n"] * es, flops=3 * case["n"])
    T, V = case["T"], case["V"]
    keep = 1.0 - case.get("mask", 0.0)
    if kind == "lm_head":
        d = case["d"]
        out = 2 if case["api"] == "autograd" else 4
        return dict(bytes=(T + V) * d * (2 + out) + 30 * T, flops=6 * T * d * V)
    es = 4 if case["dtype"] == "f32" else 2
    if kind == "logprob":
        return dict(bytes=T * V * es + T * (16 + (4 if case["versions"] > 1 else 0)), flops=3 * T * V)
    if kind == "shard":           # the statistics need the whole row before any gradient
        Vs = V // case["P"]
        return dict(bytes=2 * T * Vs * es + T * (60 + 4 * case["P"]), flops=8 * T * Vs)
    wr = 1.0 if case.get("grads", True) else 0.0
    tok = 30 + (12 if kind == "step" else 0)
    return dict(bytes=int(T * V * es * (keep + wr)) + T * tok, flops=5 * T * V)


def tolerance(case):
    kind = case["kind"]
    if kind == "ewma":
        # one rounding of each element: a 32-bit fused or unfused sum, or one bf16 last place
        return dict(rel=4e-7, max=4e-6) if case["dtype"] == "f32" else dict(rel=8e-3, max=2e-2)
    if kind == "lm_head":
        # gradients through a bf16 G; whole decisions are kept off their bounds
        return dict(rel=1e-2, max=1e-1, differ=1e-3)
    if kind == "logprob":
        return dict(rel=1e-6, max=1e-5)
    if case["dtype"] == "f32":
        return dict(rel=4e-6, max=4e-5, differ=1e-3)
    if kind == "loss" and not case["grads"]:
        return dict(rel=4e-6, max=4e-5, differ=1e-3)
    # bf16 gradients, two roundings where autograd scales them
    return dict(rel=8e-3, max=2e-2, differ=1e-3)


# ------------------------------------------------------------------ 64-bit values
def _token_math(s, lp, ref):
    """Per-token loss, weight and scale of the decoupled objective (mask_weight, token mean)."""
    mu = s["lp_mu"].double()
    lr = 0.5 * mu + 0.5 * lp if ref == "log_linear" else s["lp_ref"].double()
    A = s["adv"].double()
    m = s["mask"] != 0
    r_s, r_d = torch.exp(lp - lr), torch.exp(lr - mu)
    band = (r_d >= BAND[0]) & (r_d <= BAND[1])
    lo, hi = 1 - EPS[0], 1 + EPS[1]
    ppo = torch.where(A >= 0, r_s <= hi, r_s >= lo)
    wd = torch.where(band, r_d, torch.zeros_like(r_d))
    loss_tok = -wd * torch.minimum(r_s * A, r_s.clamp(lo, hi) * A)
    ts = s["tscale"].double() if "tscale" in s else torch.ones_like(A)
    sc = ts / max(1, int(m.sum()))
    zero = torch.zeros_like(A)
    w = torch.where(m & band & ppo, sc * wd * r_s * A, zero)
    loss_tok = torch.where(m, loss_tok, zero)
    return dict(loss=(sc * loss_tok).sum()[None], loss_tok=loss_tok,
                logp=torch.where(m, lp, zero)), w


def _dlogits(z, lse, w, ids, cols=None):
    """w (softmax - onehot) for the columns of z, which start at column 0."""
    T, V = z.shape
    d = torch.empty(T, V, dtype=torch.float64, device=DEV)
    n = max(1, _rows(T, V) // 2)
    for a in range(0, T, n):
        b = min(T, a + n)
        d[a:b] = torch.exp(z[a:b].double() - lse[a:b, None]).mul_(w[a:b, None])
    own = ids < V
    d[own.nonzero()[:, 0], ids[own]] -= w[own]
    return d


def _lse(z):
    T, V = z.shape
    n = max(1, _rows(T, V) // 2)
    return torch.cat([torch.logsumexp(z[a:a + n].double(), dim=1) for a in range(0, T, n)])


def _ewma(x, x0):
    """The proxy after one step from w = 1: w' = 1 + beta, x / w' + (beta / w') x0."""
    beta = WINDOW / (WINDOW + 2.0)
    return x.double() / (1.0 + beta) + beta / (1.0 + beta) * x0.double()


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "ewma":
        return dict(x=_ewma(s["x"], s["x0"]), w=None, count=None)
    if kind == "logprob":
        rows = torch.arange(case["T"], device=DEV)
        ver = s["ver"].long() if "ver" in s else torch.zeros_like(rows)
        lse = torch.empty(case["T"], dtype=torch.float64, device=DEV)
        zy = torch.empty_like(lse)
        for v, z in enumerate(s["mats"]):
            at = rows[ver == v]
            for c in at.split(max(1, _rows(case["T"], case["V"]) // 2)):
                lse[c] = torch.logsumexp(z[c].double(), dim=1)
            zy[at] = z[at, s["ids"][at]].double()
        return dict(logp=zy - lse, lse=lse)
    if kind == "shard":
        z, ids = s["shard"], s["ids"]
        own = _lse(z)
        g = s["gathered"].double()
        g[0] = own
        lse = torch.logsumexp(g, dim=0)
        mine = ids < z.shape[1]
        zy = s["zy_others"].double()
        zy[mine] = z[mine.nonzero()[:, 0], ids[mine]].double()
        out, w = _token_math(s, zy - lse, "given")
        return dict(out, flags=None, stats=None, shard_lse=own, zy=zy, lse=lse,
                    dlogits=_dlogits(z, lse, w, ids))
    if kind == "lm_head":
        h, wt, ids = s["hidden"].double(), s["weight"].double(), s["ids"]
        T, V = case["T"], case["V"]
        z = h @ wt.T
        lse = _lse(z)
        out, w = _token_math(s, z.gather(1, ids[:, None])[:, 0] - lse, "given")
        z = _dlogits(z, lse, w, ids)
        dh, dw = z @ wt, z.T.contiguous() @ h
        out.update(flags=None, stats=None, dhidden=dh, dweight=dw)
        if case["api"] == "autograd":
            out = dict(loss=out["loss"][0], logp=out["logp"], stats=None, dhidden=dh * ACCUM,
                       dweight=dw * ACCUM)
        return out
    z, ids = s["z"], s["ids"]
    lse = _lse(z)
    lp = z.gather(1, ids[:, None])[:, 0].double() - lse
    out, w = _token_math(s, lp, case.get("ref", "given"))
    want = case.get("grads", True)
    out.update(flags=None, stats=None, dlogits=_dlogits(z, lse, w, ids) if want else None)
    if kind == "autograd":
        return dict(loss=out["loss"][0], logp=out["logp"], stats=None, dlogits=out["dlogits"].mul_(ACCUM))
    if kind == "step":
        out["proxy"] = dict(x=_ewma(s["lp_ref"], s["x0"]), w=None, count=None)
    return out
