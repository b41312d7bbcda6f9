"""Performance cases of the ASR-KF-EGR decode path.

Every case is one batch of requests served on a context that is kept, as a
serving program does it: the context is reset, every (layer, sequence) gets its
prompt's K/V (asrkf_prefill), then `steps` tokens are decoded, each with
asrkf_decode_step for every layer and asrkf_restore with the step's logits, and
the counters are read at the end (asrkf_stats).  The queries, new K/V rows,
prompts and logits are what the model around the path would produce; they are
made on the GPU beforehand.

Inputs follow the repository's heavy-hitter recipe: per (layer, sequence, KV
head) a signed coordinate axis; a heavy hitter's key has +-beta there, other
keys a small value; everything else is N(0, 1); queries lie on the axis plus
small noise.  Every score then stays clear of tau, so freeze decisions are the
same for any order of summation.  Logits are N(0, sigma); at planted steps they
are nearly flat, which triggers the recovery ladder.
"""
import math
import random

import numpy as np
import torch

import paper_2512_11221_amd as A

# name, layers, batch, q heads, KV heads, head dim, storage type, prompt length
# range (per sequence, drawn from len_seed), decode steps, window K, Eq. 3
# softness k, vocabulary, heavy-hitter fraction, first flat-logits step (0: none)
# and their number, and the options of the context
BASE = {"layers": 1, "batch": 1, "q_heads": 32, "kv_heads": 8, "head_dim": 128, "dtype": "bf16",
        "ctx_lo": 8192, "ctx_hi": 8192, "len_seed": 1, "steps": 48, "window": 128, "k_soft": 2.0,
        "vocab": 128256, "f_hh": 0.35, "flat_at": 0, "flat_n": 0, "relevance": "abs",
        "scope": "layer", "history_W": 0, "candidates": "outside", "spill_min_D": 0}


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    return [
        # the repository's smallest configuration: fp32 rows of 64, one short
        # sequence; every step is a handful of launches (latency)
        _case("tiny-f32-b1-ctx512", q_heads=8, kv_heads=2, head_dim=64, dtype="f32", ctx_lo=512,
              ctx_hi=512, steps=64, window=32, vocab=1024, flat_at=40, flat_n=3),
        # one layer of the LLaMA-3-8B shape, one sequence of 8k: the repository's
        # single-layer configuration
        _case("8b-1layer-b1-ctx8k", steps=64),
        # a whole 32-layer model serving one user at a few thousand tokens
        # (odd length): interactive decode, launches and fixed costs count
        _case("8b-32layer-b1-ctx4k", layers=32, ctx_lo=4093, ctx_hi=4093, steps=32),
        # the repository's headline configuration: 32 layers, 8 sequences of 32k
        _case("8b-32layer-b8-ctx32k", layers=32, batch=8, ctx_lo=32768, ctx_hi=32768, steps=48),
        # the repository's ragged batch: 64 sequences of 2k to 32k
        _case("8b-ragged-b64", batch=64, ctx_lo=2048, ctx_hi=32768, steps=32),
        # a serving batch of short chats at a vocabulary that is no multiple of 4
        _case("8b-8layer-b32-short", layers=8, batch=32, ctx_lo=128, ctx_hi=2048, steps=32,
              vocab=50257),
        # wide query groups (64 q over 8 KV heads)
        _case("64q8kv-8layer-b8-ctx16k", layers=8, batch=8, q_heads=64, ctx_lo=16384, ctx_hi=16384,
              steps=24),
        # rows of 256
        _case("d256-4layer-b4-ctx8k", layers=4, batch=4, q_heads=16, kv_heads=8, head_dim=256,
              ctx_lo=7000, ctx_hi=8192, steps=32, vocab=32000),
        # plain multi-head attention (one query head per KV head)
        _case("mha-4layer-b4-ctx4k", layers=4, batch=4, q_heads=32, kv_heads=32, ctx_lo=3000,
              ctx_hi=4096, steps=32, vocab=32000),
        # relevance by attention weight instead of Eq. 2
        _case("softmax-4layer-b4-ctx8k", layers=4, batch=4, ctx_lo=8192, ctx_hi=8192, steps=32,
              relevance="softmax"),
        # token-global states with a finite history window, and a recovery ladder run
        _case("token-scope-8layer-b2-ctx6k", layers=8, batch=2, ctx_lo=5000, ctx_hi=6001, steps=40,
              k_soft=1.0, scope="token", history_W=16, flat_at=25, flat_n=3),
        # spill mode: frozen rows leave for the host store, one long sequence,
        # recovery ladder run
        _case("spill-b1-ctx32k", ctx_lo=32768, ctx_hi=32768, steps=48, k_soft=1.0, spill_min_D=2,
              flat_at=30, flat_n=3),
    ]


# head layouts and storage types that the library serves: (q, kv, dim, type)
LAYOUTS = [(8, 2, 64, "f32"), (32, 8, 128, "bf16"), (32, 8, 128, "bf16"), (32, 8, 128, "bf16"),
           (64, 8, 128, "bf16"), (32, 4, 128, "bf16"), (16, 8, 256, "bf16"), (32, 32, 128, "bf16"),
           (32, 16, 128, "bf16"), (16, 2, 64, "bf16"), (8, 8, 128, "f32")]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    hq, hkv, d, dtype = rng.choice(LAYOUTS)
    row = 2 * hkv * d * (2 if dtype == "bf16" else 4)
    c = dict(BASE, q_heads=hq, kv_heads=hkv, head_dim=d, dtype=dtype, layers=_log_int(rng, 1, 32),
             batch=_log_int(rng, 1, 64), steps=rng.randint(16, 48), len_seed=rng.randrange(1 << 20),
             window=_log_int(rng, 16, 256), k_soft=rng.choice([1.0, 2.0]),
             vocab=rng.choice([1024, 32000, 50257, 128256, _log_int(rng, 1000, 150000)]),
             f_hh=round(rng.uniform(0.2, 0.5), 3))
    # prompts: at most 4 GiB of cache in all
    most = min(32768, (4 << 30) // (row * c["layers"] * c["batch"]))
    c["ctx_hi"] = _log_int(rng, min(256, most), most)
    c["ctx_lo"] = c["ctx_hi"] if rng.random() < 0.3 else max(64, int(c["ctx_hi"] * rng.uniform(0.1, 1)))
    c["ctx_lo"] = min(c["ctx_lo"], c["ctx_hi"])
    if rng.random() < 0.4:
        c.update(flat_at=rng.randint(8, 14), flat_n=rng.randint(1, 4))
    option = rng.random()
    if option < 0.15 and c["ctx_hi"] >= 256:
        c["relevance"] = "softmax"
        c["ctx_lo"] = max(256, c["ctx_lo"])
    elif option < 0.3:
        c["scope"] = "token"
    elif option < 0.4:
        # one sequence or a few: the host store is pinned memory
        c.update(spill_min_D=2, batch=min(c["batch"], 4), layers=min(c["layers"], 2))
    if rng.random() < 0.3:
        c["history_W"] = rng.choice([8, 16, 32, 64])
    return c


def _lengths(c):
    r = random.Random(c["len_seed"])
    return [r.randint(c["ctx_lo"], c["ctx_hi"]) for _ in range(c["batch"])]


def _flat(c, t):
    return c["flat_at"] > 0 and c["flat_at"] <= t < c["flat_at"] + c["flat_n"]


def _sigma(c):
    return 3.0 if c["vocab"] >= 20000 else 2.0


def _spike(c):
    # between the entropy of N(0, sigma) logits (ln V - sigma^2 / 2) and of flat ones (ln V)
    return math.log(c["vocab"]) - _sigma(c) ** 2 / 4


def _tau(c):
    # softmax relevance: cold tokens get about 0.17 / n of the attention, hot ones over 0.6 / n
    return 0.5 if c["relevance"] == "abs" else 0.33 / (0.5 * (c["ctx_lo"] + c["ctx_hi"]))


class State:
    """What a serving program holds: the context, the prompts' K/V, and the
    tensors of each step."""

    def __init__(self):
        self.ctx = None

    def __del__(self):
        if self.ctx:
            A.asrkf_destroy(self.ctx)
            self.ctx = None


def _inputs(c, seed):
    """Prompts, per-step q / k / v and logits, on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    L, B, Hq, Hkv, D, N = (c[k] for k in ("layers", "batch", "q_heads", "kv_heads", "head_dim", "steps"))
    G = Hq // Hkv
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    dev = {"device": "cuda"}
    plen = _lengths(c)
    top = max(plen)
    soft = c["relevance"] == "softmax"
    root = math.sqrt(D / 128)
    axis = torch.randint(0, D, (L, B, Hkv), generator=g, **dev)
    sign = (torch.randint(0, 2, (L, B, Hkv), generator=g, **dev) * 2 - 1).float()

    def keys(shape, l, per_seq):
        # shape [*, B or one sequence, n, Hkv, D]; the axis entries set as the recipe says
        x = torch.randn(shape, generator=g, dtype=dt, **dev)
        n = shape[:-1]
        hot = torch.rand(n[:-1], generator=g, **dev) < c["f_hh"]
        u = torch.rand(n, generator=g, **dev)
        beta = (32 + 32 * u) if soft else (8 + 56 * u)
        a, s = per_seq
        at = a.expand(n).unsqueeze(-1)
        small = x.gather(-1, at).squeeze(-1).float() * 2.0 ** -4
        x.scatter_(-1, at, torch.where(hot.unsqueeze(-1), s * beta, small).to(dt).unsqueeze(-1))
        return x

    prompts = []
    for l in range(L):
        a, s = axis[l].view(B, 1, Hkv), sign[l].view(B, 1, Hkv)
        K = keys((B, top, Hkv, D), l, (a, s))
        V = torch.randn((B, top, Hkv, D), generator=g, dtype=dt, **dev)
        prompts.append((K, V))
    a, s = axis.view(1, L, B, Hkv), sign.view(1, L, B, Hkv)
    kn = keys((N, L, B, Hkv, D), None, (a, s))
    vn = torch.randn((N, L, B, Hkv, D), generator=g, dtype=dt, **dev)
    q = torch.randn((N, L, B, Hq, D), generator=g, **dev) * 2.0 ** -13
    u = torch.rand((N, L, B, Hq), generator=g, **dev)
    alpha = (0.5 + 0.25 * u) * root if soft else 0.2 + 0.1 * u
    aq = axis.repeat_interleave(G, dim=2).view(1, L, B, Hq).expand(N, L, B, Hq).unsqueeze(-1)
    sq = sign.repeat_interleave(G, dim=2).view(1, L, B, Hq)
    q.scatter_add_(-1, aq, (alpha * sq).unsqueeze(-1))
    q = q.to(dt)
    logits = []
    for t in range(1, N + 1):
        x = torch.randn((B, c["vocab"]), generator=g, **dev)
        logits.append(x * (0.1 if _flat(c, t) else _sigma(c)))
    return plen, prompts, kn, vn, q, logits


def prepare(case, seed):
    c = case
    s = State()
    s.plen, prompts, kn, vn, q, s.logits = _inputs(c, seed)
    L, B, N = c["layers"], c["batch"], c["steps"]
    s.prompts = [[(K[b], V[b]) for b in range(B)] for K, V in prompts]
    s.out = torch.empty((N, L, B, c["q_heads"], c["head_dim"]), device="cuda")
    s.rows = [[(q[t, l], kn[t, l], vn[t, l], s.out[t, l]) for l in range(L)] for t in range(N)]
    s.monitor = B <= 4
    s.spill = c["spill_min_D"] > 0
    s.ctx = A.asrkf_init(A.make_config(
        L, B, c["q_heads"], c["kv_heads"], c["head_dim"], max(s.plen) + N, c["window"], _tau(c),
        c["k_soft"], c["vocab"], entropy_spike=_spike(c), dtype=c["dtype"],
        spill_min_D=c["spill_min_D"], history_W=c["history_W"], relevance=c["relevance"],
        scope=c["scope"], candidates=c["candidates"]))
    return s


def run(state):
    s, ctx = state, state.ctx
    stream = torch.cuda.current_stream().cuda_stream
    A.asrkf_reset(ctx)
    for l, layer in enumerate(s.prompts):
        for b, (K, V) in enumerate(layer):
            A.asrkf_prefill(ctx, l, b, K, V, s.plen[b], stream)
    for layers, logits in zip(s.rows, s.logits):
        for l, (q, k, v, out) in enumerate(layers):
            A.asrkf_decode_step(ctx, l, q, k, v, out, stream)
        A.asrkf_restore(ctx, logits, A.AUTO, stream)
    st = A.asrkf_stats(ctx)
    keys = ["step", "total_positions", "active_positions", "attended_total", "rr_requests"]
    if s.spill:
        keys += ["rows_to_host", "rows_from_host", "rows_released", "rows_reused"]
    got = {"out": s.out, "counters": np.array([st[k] for k in keys] + st["recoveries"], dtype=np.int64)}
    if s.monitor:                   # few sequences: their entropy monitors are read too
        seqs = [A.asrkf_get_seq(ctx, b) for b in range(len(s.plen))]
        got["entropy"] = np.array([x["entropy"] for x in seqs], dtype=np.float32)
        got["pmax"] = np.array([x["pmax"] for x in seqs], dtype=np.float32)
        got["ladder"] = np.array([[x["escalation"], x["level"]] for x in seqs], dtype=np.int64)
    return got


def _levels(spikes):
    esc, out = 0, []
    for x in spikes:
        esc = esc + 1 if x else 0
        out.append(min(esc, 3))
    return out


def _attended(c):
    """Expected attended tokens summed over steps, one layer: the heavy hitters
    always, the cold tokens on the schedule of one always-flagged token (the
    tokens still inside the window attend always)."""
    total, unfreeze, seen = 0.0, 0, []
    plen = _lengths(c)
    levels = _levels(_flat(c, t) for t in range(1, c["steps"] + 1))
    for t in range(1, c["steps"] + 1):
        n = sum(p + t for p in plen)
        cold = sum(max(0, p + t - c["window"]) for p in plen) * (1 - c["f_hh"])
        total += n
        if unfreeze > t:
            total -= cold
        else:
            seen.append(t)
            W = c["history_W"]
            count = len([x for x in seen if W == 0 or x > t - W])
            d = int(math.sqrt(count) / c["k_soft"])
            if d >= 1:
                unfreeze = t + d
        if levels[t - 1] == 3 or (levels[t - 1] == 1 and unfreeze > t + 2):
            unfreeze = min(unfreeze, t + 1)
    return total


def work(case):
    c = case
    esz = 2 if c["dtype"] == "bf16" else 4
    row = 2 * c["kv_heads"] * c["head_dim"] * esz           # K and V of one token
    att = _attended(c) * c["layers"]
    prompt = sum(_lengths(c)) * c["layers"] * row
    per_step = c["layers"] * c["batch"] * (c["q_heads"] * c["head_dim"] * (esz + 4) + 2 * row)
    by = 2 * prompt + att * row + c["steps"] * (per_step + 4 * c["batch"] * c["vocab"])
    if c["spill_min_D"]:
        # every cold token's rows leave once
        by += 2 * (1 - c["f_hh"]) * prompt
    return {"bytes": by, "flops": att * 4 * c["q_heads"] * c["head_dim"]}


def tolerance(case):
    # bf16 / fp32 rows, sums and softmax in 32 bits: against 64 bits the outputs
    # are 1.2e-7 (short prompts) to 3.3e-7 (32k) off in the 2-norm, the entropies up to
    # 2e-7; two correct implementations differ by up to twice that, and this is about
    # four times it.  Whole values are decided on scores clear of tau: the same.
    return {"rel": 3e-6, "max": 1e-4, "differ": 0.0}


def exact(case, seed):
    """The same decode in 64 bits: the cache masked by each token's unfreeze
    step, one sequence after the other."""
    c = case
    L, B, Hq, Hkv, D, N = (c[k] for k in ("layers", "batch", "q_heads", "kv_heads", "head_dim", "steps"))
    plen = _lengths(c)
    # bytes of 64-bit K/V walked; beyond this it would take more than about 20 s
    if sum(plen) * L * N * Hkv * D * 16 > 6e12:
        return None
    plen, prompts, kn, vn, q, logits = _inputs(c, seed)
    G, W, tau = Hq // Hkv, c["history_W"], _tau(c)
    # entropy monitor and the ladder
    H = torch.empty((N, B), dtype=torch.float64, device="cuda")
    pm = torch.empty_like(H)
    for t in range(N):
        p = torch.log_softmax(logits[t].double(), dim=-1)
        H[t] = -(p.exp() * p).sum(-1)
        pm[t] = p.max(-1).values.exp()
    spikes = (H > _spike(c)).cpu()
    out = torch.empty((N, L, B, Hq, D), dtype=torch.float64, device="cuda")

    def cache(l, b):
        P = plen[b]
        K = torch.cat([prompts[l][0][b, :P].double(), kn[:, l, b].double()])
        V = torch.cat([prompts[l][1][b, :P].double(), vn[:, l, b].double()])
        return K.permute(1, 2, 0).contiguous(), V.permute(1, 0, 2).contiguous()

    def attend(KV, l, b, t, on, n):
        # [Hkv, G, n] products, the attention over the active positions and the scores
        x = torch.matmul(q[t - 1, l, b].double().view(Hkv, G, D), KV[0][:, :, :n])
        p = torch.softmax((x / math.sqrt(D)).masked_fill(~on, -math.inf), dim=-1)
        out[t - 1, l, b] = torch.matmul(p, KV[1][:, :n]).reshape(Hq, D)
        return (x.abs() if c["relevance"] == "abs" else p).sum((0, 1)) / Hq

    for b in range(B):
        P = plen[b]
        levels = _levels(bool(spikes[t, b]) for t in range(N))
        pos = torch.arange(P + N, device="cuda")
        groups = [list(range(L))] if c["scope"] == "token" else [[l] for l in range(L)]
        for layers in groups:
            KVs = [cache(l, b) for l in layers]
            U = torch.zeros(P + N, dtype=torch.int64, device="cuda")
            seen = torch.zeros((N + 1, P + N), dtype=torch.int64, device="cuda")
            for t in range(1, N + 1):
                n = P + t
                on = U[:n] <= t
                s = sum(attend(KV, l, b, t, on, n) for KV, l in zip(KVs, layers)) / len(layers)
                edge = n - c["window"]
                where = pos[:n] < edge if c["candidates"] == "outside" else pos[:n] >= edge
                low = on & where & (s < tau)
                seen[t, :n] = low
                count = seen[(0 if W == 0 else max(0, t - W + 1)):t + 1, :n].sum(0)
                d = (count.double().sqrt() / c["k_soft"]).floor().long()
                u = torch.where(low & (d >= 1), t + d, U[:n])
                level = levels[t - 1]
                if level == 1:
                    u = torch.where(u > t + 2, t + 1, u)
                elif level == 2:
                    u = torch.where((pos[:n] >= n - 4 * c["window"]) & (u > t + 1), t + 1, u)
                elif level == 3:
                    u = torch.where(u > t + 1, t + 1, u)
                U[:n] = u
    got = {"out": out, "counters": None}
    if B <= 4:
        got.update(entropy=H[-1].cpu().numpy(), pmax=pm[-1].cpu().numpy(), ladder=None)
    return got
