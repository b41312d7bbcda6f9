"""Attention tiles and their split over workgroups, at the sizes where they can
go wrong: lists that end at, before and after a tile's edge (16, 32 or 64
tokens by row size) and a workgroup's (eight tiles), the appended token alone in
a tile, empty lists, batches planned in registers (up to 64 sequences) and in
LDS (more), workgroups that take one KV head and workgroups that take eight,
pieces longer than the room for their relevance values, values that are not
finite, and prompts whose rows are not 16-byte aligned.

Bound on the outputs: K, V and q are exact in both implementations, so what
differs is fp32 rounding.  A score of up to 256 products carries at most 256
roundings of 2^-24 relative to its largest partial sum, the weights inherit its
absolute error, and the sums over the list add about sqrt(n) roundings: 1e-5 of
the values' range (|v| < 3.5) leaves more than a factor of ten."""
import math

import numpy as np
import pytest

from synth import gen
from tests import _harness as H

pytestmark = pytest.mark.gpu

OUT_TOL = 1e-5 * 3.5


@pytest.fixture(scope="module", autouse=True)
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11221_amd as A
    A.load()
    return torch


def _parity(w):
    inp = H.Inputs(w)
    inst = [(l, b) for l in range(w.n_layers) for b in range(w.batch)]
    g, _, _ = H.run_gpu(w, inp, inst)
    o = H.run_oracle(w, inp, inst)
    worst = max(H.compare_instance(g[k], o[k]) for k in inst)
    assert worst <= OUT_TOL, worst


LAYOUTS = {
    "bf16-128-g4": dict(n_q_heads=32, n_kv_heads=8, head_dim=128, dtype="bf16"),
    "bf16-128-g8": dict(n_q_heads=16, n_kv_heads=2, head_dim=128, dtype="bf16"),
    "bf16-64-g2": dict(n_q_heads=8, n_kv_heads=4, head_dim=64, dtype="bf16"),
    "bf16-64-g1": dict(n_q_heads=32, n_kv_heads=32, head_dim=64, dtype="bf16"),
    "bf16-256-g8": dict(n_q_heads=8, n_kv_heads=1, head_dim=256, dtype="bf16"),
    "bf16-256-g2": dict(n_q_heads=8, n_kv_heads=4, head_dim=256, dtype="bf16"),
    "f32-64-g4": dict(n_q_heads=8, n_kv_heads=2, head_dim=64, dtype="f32"),
    "f32-64-g8": dict(n_q_heads=8, n_kv_heads=1, head_dim=64, dtype="f32"),
    "f32-128-g1": dict(n_q_heads=4, n_kv_heads=4, head_dim=128, dtype="f32"),
    "f32-128-g2": dict(n_q_heads=8, n_kv_heads=4, head_dim=128, dtype="f32"),
}


@pytest.mark.parametrize("layout", sorted(LAYOUTS))
def test_tile_and_workgroup_edges(layout):
    """One batch of all edge lengths; the four steps move each across its edge.
    Every out-of-window token freezes, so the lists shrink again."""
    lay = LAYOUTS[layout]
    tile = 8192 // (lay["head_dim"] * (2 if lay["dtype"] == "bf16" else 4))
    w = gen.Workload(name=f"tiles-{layout}", seed=gen.SEED + 201, n_layers=1, batch=8,
                     prefill=[0, 1, tile - 3, tile - 1, tile, 8 * tile - 2, 8 * tile + 1, 20 * tile + 5],
                     steps=5, window_K=3, tau=math.inf, k_soft=0.5, vocab=64, logit_sigma=1.0,
                     recipe="gauss", **lay)
    _parity(w)


@pytest.mark.parametrize("relevance", ["abs", "softmax"])
@pytest.mark.parametrize("scope", ["layer", "token"])
@pytest.mark.parametrize("batch", [64, 65, 130])
def test_many_sequences(batch, scope, relevance):
    """64 sequences are planned in registers, more in LDS; with 8 KV heads they
    give a workgroup two, four and eight heads of a sequence together."""
    w = gen.Workload(name=f"tiles-b{batch}-{scope}-{relevance}", seed=gen.SEED + 202, n_layers=2,
                     batch=batch, n_q_heads=16, n_kv_heads=8, head_dim=64, dtype="bf16",
                     prefill=[900 if b == 3 else (0 if b % 7 == 2 else 5 + 13 * b % 90) for b in range(batch)],
                     steps=4, window_K=4, tau=math.inf, k_soft=0.5, vocab=64, logit_sigma=1.0,
                     recipe="gauss", scope=scope, relevance=relevance)
    _parity(w)


def test_logits_beyond_the_room():
    """Eight query heads' logits (softmax reading) fill the room for kept values
    after 32 tiles; one sequence of 66.2k tokens gives every workgroup 33."""
    w = gen.Workload(name="tiles-room", seed=gen.SEED + 203, n_layers=1, batch=1, n_q_heads=64,
                     n_kv_heads=8, head_dim=64, dtype="bf16", prefill=[66200], steps=2, window_K=8,
                     tau=math.inf, k_soft=0.5, vocab=64, logit_sigma=1.0, recipe="gauss",
                     relevance="softmax")
    _parity(w)


@pytest.mark.parametrize("batch,n", [(66, 8700), (8, 72000)])
def test_relevance_beyond_the_room(gpu, batch, n):
    """Long pieces of workgroups that take eight KV heads: their summed relevance
    is stored in chunks.  Every token scoring below tau must freeze (k = 1/4
    freezes at the first detection) and no other, against scores in 64 bits;
    tokens within 1e-3 of tau are left out (a score of 64 products of |z| < 3.5
    carries less than 1e-4 of rounding)."""
    torch = gpu
    import paper_2512_11221_amd as A
    Hq, Hkv, D = 8, 8, 64
    g = torch.Generator(device="cuda").manual_seed(7)
    tau = 6.0
    cfg = A.make_config(1, batch, Hq, Hkv, D, n + 4, 16, tau, 0.25, 16, dtype="bf16")
    ctx = A.asrkf_init(cfg)
    try:
        K = torch.randn((batch, n + 1, Hkv, D), generator=g, device="cuda", dtype=torch.bfloat16)
        V = torch.randn((batch, n + 1, Hkv, D), generator=g, device="cuda", dtype=torch.bfloat16)
        q = torch.randn((batch, Hq, D), generator=g, device="cuda", dtype=torch.bfloat16)
        out = torch.empty((batch, Hq, D), device="cuda")
        for b in range(batch):
            A.asrkf_prefill(ctx, 0, b, K[b], V[b], n)
        A.asrkf_decode_step(ctx, 0, q, K[:, n].contiguous(), V[:, n].contiguous(), out)
        A.asrkf_restore(ctx, None, A.NONE)
        for b in list(range(0, batch, 9)) + [batch - 1]:
            x = (K[b].double() * q[b].double()).sum(-1)                     # [n + 1][heads]
            ref = (torch.softmax(x / math.sqrt(D), 0).unsqueeze(-1) * V[b].double()).sum(0)
            assert float((out[b].double() - ref).abs().max()) <= OUT_TOL
            s = x.abs().mean(1).cpu().numpy()
            st = A.asrkf_get_state(ctx, 0, b, n + 4)
            want = (s < tau) & (np.arange(n + 1) < n + 1 - 16)
            clear = np.abs(s - tau) > 1e-3
            np.testing.assert_array_equal(st["frozen"][clear], want[clear])
            assert 0.05 < want.mean() < 0.95
    finally:
        A.asrkf_destroy(ctx)


@pytest.mark.parametrize("layout", ["bf16-128-g4", "bf16-128-g8", "bf16-64-g2", "bf16-64-g1", "bf16-256-g8", "f32-64-g4"])
def test_infinite_values(gpu, layout):
    """An infinity in a value row reaches the dims it sits in, with its sign, and
    no others; two of opposite sign give NaN there."""
    torch = gpu
    import paper_2512_11221_amd as A
    lay = LAYOUTS[layout]
    Hq, Hkv, D = lay["n_q_heads"], lay["n_kv_heads"], lay["head_dim"]
    dt = torch.bfloat16 if lay["dtype"] == "bf16" else torch.float32
    n = 300
    g = torch.Generator(device="cuda").manual_seed(9)
    ctx = A.asrkf_init(A.make_config(1, 1, Hq, Hkv, D, n + 2, 16, 0.0, 2.0, 16, dtype=lay["dtype"]))
    try:
        K = torch.randn((n + 1, Hkv, D), generator=g, device="cuda", dtype=dt) * 0.1
        V = torch.randn((n + 1, Hkv, D), generator=g, device="cuda", dtype=dt)
        V[7, 0, 3] = math.inf
        V[200, 0, 5] = -math.inf
        V[20, 0, 9] = math.inf
        V[290, 0, 9] = -math.inf
        q = torch.randn((1, Hq, D), generator=g, device="cuda", dtype=dt)
        out = torch.empty((1, Hq, D), device="cuda")
        A.asrkf_prefill(ctx, 0, 0, K, V, n)
        A.asrkf_decode_step(ctx, 0, q, K[n:].contiguous(), V[n:].contiguous(), out)
        G = Hq // Hkv
        o = out[0].cpu().numpy()
        assert (o[:G, 3] == math.inf).all() and (o[:G, 5] == -math.inf).all() and np.isnan(o[:G, 9]).all()
        rest = np.delete(o[:G], [3, 5, 9], axis=1)
        assert np.isfinite(rest).all() and np.isfinite(o[G:]).all()
    finally:
        A.asrkf_destroy(ctx)


@pytest.mark.parametrize("offset", [0, 1, 2, 8])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_prompt_alignment(gpu, dtype, offset):
    """Prompt rows at any element alignment land in the cache as they are: the
    outputs equal those of an aligned copy, bit for bit."""
    torch = gpu
    import paper_2512_11221_amd as A
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    n, Hkv, D = 137, 4, 64
    g = torch.Generator(device="cuda").manual_seed(11)
    flat = torch.randn((2, n * Hkv * D + 8), generator=g, device="cuda", dtype=dt)
    kv = [x[offset:offset + n * Hkv * D] for x in flat]
    q = torch.randn((1, 8, D), generator=g, device="cuda", dtype=dt)
    new = torch.randn((2, 1, Hkv, D), generator=g, device="cuda", dtype=dt)
    outs = []
    for k, v in (kv, [x.clone() for x in kv]):
        ctx = A.asrkf_init(A.make_config(1, 1, 8, Hkv, D, n + 2, 16, 0.5, 2.0, 16, dtype=dtype))
        try:
            out = torch.empty((1, 8, D), device="cuda")
            A.asrkf_prefill(ctx, 0, 0, k, v, n)
            A.asrkf_decode_step(ctx, 0, q, new[0], new[1], out)
            outs.append(out.cpu().numpy())
        finally:
            A.asrkf_destroy(ctx)
    np.testing.assert_array_equal(outs[0], outs[1])


def _one_step(gpu, layout, batch, n, poison):
    """One step over `batch` sequences of n prompt tokens; poison(K) edits the
    keys [batch][n + 1][Hkv][D] first (the last row is the new token's).  Query
    entries 5 are positive.  Returns q, K, V and the output, in 64 bits."""
    torch = gpu
    import paper_2512_11221_amd as A
    lay = LAYOUTS[layout]
    Hq, Hkv, D = lay["n_q_heads"], lay["n_kv_heads"], lay["head_dim"]
    dt = torch.bfloat16 if lay["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(17)
    K = torch.randn((batch, n + 1, Hkv, D), generator=g, device="cuda", dtype=dt)
    V = torch.randn((batch, n + 1, Hkv, D), generator=g, device="cuda", dtype=dt)
    q = torch.randn((batch, Hq, D), generator=g, device="cuda", dtype=dt)
    q[..., 5] = q[..., 5].abs() + 0.125
    poison(K)
    out = torch.empty((batch, Hq, D), device="cuda")
    ctx = A.asrkf_init(A.make_config(1, batch, Hq, Hkv, D, n + 2, 16, 0.0, 2.0, 16, dtype=lay["dtype"]))
    try:
        for b in range(batch):
            A.asrkf_prefill(ctx, 0, b, K[b], V[b], n)
        A.asrkf_decode_step(ctx, 0, q, K[:, n].contiguous(), V[:, n].contiguous(), out)
        return [x.double().cpu() for x in (q, K, V, out)]
    finally:
        A.asrkf_destroy(ctx)


# where the keys of KV head 0 of the last sequence are not finite: the new token
# alone in its tile; whole tiles, so that one wave or one workgroup sees nothing
# else; a single one among others
POISONED = {"new": (1, 576, [576]), "tiles": (1, 600, range(64, 256)), "first": (1, 600, range(0, 192)),
            "one": (1, 600, [10]), "batch": (66, 64, [64])}


@pytest.mark.parametrize("where", sorted(POISONED))
@pytest.mark.parametrize("layout", ["bf16-128-g4", "bf16-128-g8", "bf16-64-g1", "bf16-256-g2", "f32-64-g4"])
def test_nan_keys(gpu, layout, where):
    """A score that is no number makes its head's outputs NaN, wherever the token
    falls among the waves and workgroups, and no other head's."""
    batch, n, rows = POISONED[where]

    def poison(K):
        K[-1, list(rows), 0, 5] = math.nan
    q, K, V, out = _one_step(gpu, layout, batch, n, poison)
    G = q.shape[1] // K.shape[2]
    assert out[-1, :G].isnan().all()
    assert out[-1, G:].isfinite().all() and out[:-1].isfinite().all()


@pytest.mark.parametrize("where", sorted(POISONED))
@pytest.mark.parametrize("layout", ["bf16-128-g4", "bf16-128-g8", "bf16-64-g1", "f32-64-g4"])
def test_scores_of_minus_infinity(gpu, layout, where):
    """A score of -inf weighs nothing, also where a wave or a workgroup sees only
    such scores."""
    torch = gpu
    batch, n, rows = POISONED[where]

    def poison(K):
        K[-1, list(rows), 0, 5] = -math.inf
    q, K, V, out = _one_step(gpu, layout, batch, n, poison)
    G, D = q.shape[1] // K.shape[2], q.shape[2]
    for h in range(q.shape[1]):
        x = K[-1, :, h // G] @ q[-1, h] / math.sqrt(D)
        ref = torch.softmax(x, 0) @ V[-1, :, h // G]
        assert float((out[-1, h] - ref).abs().max()) <= OUT_TOL


@pytest.mark.parametrize("layout", ["bf16-128-g4", "bf16-128-g8", "bf16-64-g1", "bf16-256-g2", "f32-64-g4"])
def test_values_near_the_largest(gpu, layout):
    """Values of 2^125 on tokens that score 5.5 (log2 units) above everything
    before them, one such token per dimension: with weights of at most 1 every sum
    stays below 2^126.  Bound: relative, as for ordinary values."""
    torch = gpu
    import paper_2512_11221_amd as A
    lay = LAYOUTS[layout]
    Hq, Hkv, D = lay["n_q_heads"], lay["n_kv_heads"], lay["head_dim"]
    dt = torch.bfloat16 if lay["dtype"] == "bf16" else torch.float32
    n, batch = 1200, 66
    g = torch.Generator(device="cuda").manual_seed(19)
    K = torch.zeros((n + 1, Hkv, D), device="cuda")
    V = torch.randn((n + 1, Hkv, D), generator=g, device="cuda").to(dt).float()
    high = 600 + 9 * torch.arange(64, device="cuda")
    K[high, :, 0] = 5.5 * math.sqrt(D) / math.log2(math.e)
    V[high, :, torch.arange(64, device="cuda")] = 2.0 ** 125
    K, V = K.to(dt), V.to(dt)
    q = torch.zeros((batch, Hq, D), device="cuda", dtype=dt)
    q[..., 0] = 1.0
    out = torch.empty((batch, Hq, D), device="cuda")
    ctx = A.asrkf_init(A.make_config(1, batch, Hq, Hkv, D, n + 2, 16, 0.0, 2.0, 16, dtype=lay["dtype"]))
    try:
        for b in range(batch):
            A.asrkf_prefill(ctx, 0, b, K, V, n)
        new = [x[n:].expand(batch, Hkv, D).contiguous() for x in (K, V)]
        A.asrkf_decode_step(ctx, 0, q, new[0], new[1], out)
        w = torch.softmax(K[:, 0, 0].double() / math.sqrt(D), 0)
        ref = torch.einsum("n,nhd->hd", w, V.double()).repeat_interleave(Hq // Hkv, 0)
        assert float(((out.double() - ref) / ref.abs().clamp_min(1.0)).abs().max()) <= 1e-5
    finally:
        A.asrkf_destroy(ctx)


@pytest.mark.parametrize("n", [1, 33, 700, 9000])
@pytest.mark.parametrize("layout", ["bf16-64-g8", "bf16-128-g8", "bf16-256-g8"])
def test_eight_query_heads_error(gpu, layout, n):
    """Eight query heads take their weights' 24 bits in two passes.  Bound in the 2-norm: weights exact to fp32 and sums in fp32
    give about 2e-7 (measured 1.0e-7 to 1.7e-7); a weight cut to 16 bits would give
    some 1e-5 / sqrt(n), 1e-6 and more up to 100 tokens."""
    torch = gpu
    import paper_2512_11221_amd as A
    Hq, Hkv, D = {"bf16-64-g8": (16, 2, 64), "bf16-128-g8": (16, 2, 128), "bf16-256-g8": (8, 1, 256)}[layout]
    g = torch.Generator(device="cuda").manual_seed(31 + n)
    K, V = (torch.randn((n + 1, Hkv, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    q = torch.randn((1, Hq, D), generator=g, device="cuda", dtype=torch.bfloat16)
    out = torch.empty((1, Hq, D), device="cuda")
    ctx = A.asrkf_init(A.make_config(1, 1, Hq, Hkv, D, n + 2, 16, 0.0, 2.0, 16, dtype="bf16"))
    try:
        A.asrkf_prefill(ctx, 0, 0, K, V, n)
        A.asrkf_decode_step(ctx, 0, q, K[n:].contiguous(), V[n:].contiguous(), out)
        x = torch.matmul(q[0].double().view(Hkv, 8, D), K.double().permute(1, 2, 0).contiguous())
        p = torch.softmax(x / math.sqrt(D), -1)
        ref = torch.matmul(p, V.double().permute(1, 0, 2).contiguous()).view(Hq, D)
        err = float((out[0].double() - ref).norm() / ref.norm())
        print(f"{layout} n {n}: {err:.2e}")
        assert err <= 4e-7
    finally:
        A.asrkf_destroy(ctx)


@pytest.mark.parametrize("layout,batch", [
    ("bf16-64-g1", 8), ("bf16-64-g1", 16), ("bf16-64-g1", 32), ("bf16-64-g1", 64), ("bf16-64-g1", 70),
    ("bf16-128-g4", 40), ("bf16-128-g4", 100), ("bf16-128-g4", 300), ("bf16-128-g8", 200), ("bf16-256-g2", 90),
    ("f32-128-g1", 100), ("f32-64-g8", 300)])
def test_pairs_shared_by_workgroups_of_several_heads(gpu, layout, batch):
    """Ragged batches whose pairs are cut by the ranges of workgroups that take one,
    two, four or eight KV heads together: every sequence's outputs against 64 bits."""
    torch = gpu
    import paper_2512_11221_amd as A
    lay = LAYOUTS[layout]
    Hq, Hkv, D = lay["n_q_heads"], lay["n_kv_heads"], lay["head_dim"]
    dt = torch.bfloat16 if lay["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(37)
    lens = [1 + (97 * b * b + 31 * b) % 700 for b in range(batch)]
    n = max(lens)
    K, V = (torch.randn((n + 1, Hkv, D), generator=g, device="cuda", dtype=dt) for _ in range(2))
    q = torch.randn((batch, Hq, D), generator=g, device="cuda", dtype=dt)
    new = [x[n:].expand(batch, Hkv, D).contiguous() for x in (K, V)]
    out = torch.empty((batch, Hq, D), device="cuda")
    ctx = A.asrkf_init(A.make_config(1, batch, Hq, Hkv, D, n + 2, 16, 0.0, 2.0, 16, dtype=lay["dtype"]))
    try:
        for b in range(batch):
            A.asrkf_prefill(ctx, 0, b, K, V, lens[b])
        A.asrkf_decode_step(ctx, 0, q, new[0], new[1], out)
        Kd, Vd = (x.double().permute(1, 0, 2).contiguous() for x in (K, V))       # [Hkv][n + 1][D]
        x = torch.matmul(q.double().view(batch, Hkv, Hq // Hkv, D), Kd.transpose(1, 2).contiguous())
        pos = torch.arange(n + 1, device="cuda")
        off = (pos >= torch.tensor(lens, device="cuda")[:, None]) & (pos < n)     # the new token is row n
        p = torch.softmax((x / math.sqrt(D)).masked_fill(off[:, None, None], -math.inf), -1)
        ref = torch.matmul(p, Vd).view(batch, Hq, D)
        assert float((out.double() - ref).abs().max()) <= OUT_TOL * 1.5           # |v| < 5.2
    finally:
        A.asrkf_destroy(ctx)


@pytest.mark.parametrize("batch,n", [(66, 1200), (40, 900)])
def test_logits_of_several_heads_beyond_the_room(gpu, batch, n):
    """Softmax reading with four and two KV heads of eight query heads together: the
    room for kept logits is full after eight and sixteen tiles of 64 tokens, so a
    piece stores them in several chunks.  Which tokens freeze against scores in 64
    bits, without those within 1e-3 of tau (a weight carries about 1e-5 of
    relative rounding)."""
    torch = gpu
    import paper_2512_11221_amd as A
    Hq, Hkv, D = 64, 8, 64
    g = torch.Generator(device="cuda").manual_seed(41)
    tau = 1.0 / (n + 1)
    K = torch.randn((batch, n + 1, Hkv, D), generator=g, device="cuda", dtype=torch.bfloat16)
    q = torch.randn((batch, Hq, D), generator=g, device="cuda", dtype=torch.bfloat16)
    new = K[:, n].contiguous()
    out = torch.empty((batch, Hq, D), device="cuda")
    ctx = A.asrkf_init(A.make_config(1, batch, Hq, Hkv, D, n + 2, 16, tau, 0.25, 16, dtype="bf16",
                                     relevance="softmax"))
    try:
        for b in range(batch):
            A.asrkf_prefill(ctx, 0, b, K[b], K[b], n)
        A.asrkf_decode_step(ctx, 0, q, new, new, out)
        A.asrkf_restore(ctx, None, A.NONE)
        x = torch.matmul(K.double().permute(0, 2, 1, 3),                          # [B][Hkv][n + 1][G]
                         q.double().view(batch, Hkv, Hq // Hkv, D).transpose(2, 3).contiguous())
        s = (torch.softmax(x / math.sqrt(D), 2).sum((1, 3)) / Hq).cpu().numpy()
        for b in range(batch):
            st = A.asrkf_get_state(ctx, 0, b, n + 2)
            want = (s[b] < tau) & (np.arange(n + 1) < n + 1 - 16)
            clear = np.abs(s[b] - tau) > 1e-3 * tau
            np.testing.assert_array_equal(st["frozen"][clear], want[clear])
            assert 0.2 < want.mean() < 0.8
    finally:
        A.asrkf_destroy(ctx)
