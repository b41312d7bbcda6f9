"""The planes that hold the attended tokens' relevance until their verdicts: the
device memory of a context, verdicts of a step in several launches (the planes of
only some layers are kept), and a context in a device with little memory left.

A plane holds 4 bytes per cached position; a context keeps those of all layers
up to a 32nd of its K and V rows (or 256 MiB)."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11221_amd as A
    A.load()
    return torch


def _used(torch, A, **kw):
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx = A.asrkf_init(A.make_config(window_K=16, tau=0.5, k_soft=2.0, vocab=64, **kw))
    try:
        return before - torch.cuda.mem_get_info()[0]
    finally:
        A.asrkf_destroy(ctx)


@pytest.mark.parametrize("relevance", ["abs", "softmax"])
@pytest.mark.parametrize("heads", [(32, 8, 128), (32, 4, 64), (16, 2, 64)])
def test_device_memory_of_a_context(gpu, heads, relevance):
    """K and V rows, a 32nd of them (or 256 MiB) for the planes, 13 bytes of state per position
    (unfreeze step, count, flag, list entry), 16 MiB of the rest (split partials,
    small arrays, and what the allocator rounds up)."""
    import paper_2512_11221_amd as A
    Hq, Hkv, D = heads
    L, B, n = 32, 4, 65535
    rows = 2 * L * B * (n + 1) * Hkv * D * 2
    used = _used(gpu, A, n_layers=L, batch=B, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, max_ctx=n,
                 dtype="bf16", relevance=relevance)
    assert used <= rows + max(rows // 32, 256 << 20) + 13 * L * B * (n + 1) + (16 << 20)


@pytest.mark.parametrize("relevance", ["abs", "softmax"])
def test_device_memory_with_few_device_rows(gpu, relevance):
    """Spill mode's planes follow the device rows: 39 bytes per position (13 as
    above, 26 of row bookkeeping), 8 MiB of planes."""
    import paper_2512_11221_amd as A
    L, n, rows = 2, 131071, 4096
    used = _used(gpu, A, n_layers=L, batch=1, n_q_heads=32, n_kv_heads=8, head_dim=128, max_ctx=n,
                 dtype="bf16", relevance=relevance, spill_min_D=2, device_rows=rows)
    pool = 2 * L * rows * 2048
    assert used <= pool + (8 << 20) + 39 * L * (n + 1) + 8 * L * rows + (16 << 20)


# 78 MiB of planes per layer: three layers' are kept, so eight layers take the
# verdicts in launches of three, three and two layers
L, B, HQ, HKV, D, N = 8, 16, 64, 8, 64, 20000


def _inputs(torch):
    g = torch.Generator(device="cuda").manual_seed(23)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)
    return rnd(L, B, N + 1, HKV, D), rnd(L, B, N + 1, HKV, D), rnd(L, B, HQ, D)


def _context(A, scope, K, V):
    ctx = A.asrkf_init(A.make_config(L, B, HQ, HKV, D, N + 8, 16, 1.0 / (N + 1), 0.25, 16, dtype="bf16",
                                     relevance="softmax", scope=scope))
    for l in range(L):
        for b in range(B):
            A.asrkf_prefill(ctx, l, b, K[l, b], V[l, b], N)
    return ctx


def _step(A, ctx, q, k, v, out):
    for l in range(L):
        A.asrkf_decode_step(ctx, l, q[l], k[l], v[l], out[l])
    A.asrkf_restore(ctx, None, A.NONE)


@pytest.mark.parametrize("scope", ["layer", "token"])
def test_verdicts_in_several_launches(gpu, scope):
    """Which tokens freeze against scores in 64 bits (k = 1/4 freezes at the first
    detection), without those within 1e-3 of tau: a softmax weight carries about
    1e-5 of relative rounding."""
    torch = gpu
    import paper_2512_11221_amd as A
    K, V, q = _inputs(torch)
    new = [x[:, :, N].contiguous() for x in (K, V)]
    out = torch.empty((L, B, HQ, D), device="cuda")
    ctx = _context(A, scope, K, V)
    try:
        _step(A, ctx, q, new[0], new[1], out)
        s = torch.empty((L, B, N + 1), dtype=torch.float64)
        for l in range(L):
            x = torch.matmul(K[l].double().permute(0, 2, 1, 3),                 # [B][Hkv][N + 1][G]
                             q[l].double().view(B, HKV, HQ // HKV, D).transpose(2, 3).contiguous())
            s[l] = torch.softmax(x / math.sqrt(D), 2).sum((1, 3)).cpu() / HQ
        if scope == "token":
            s[:] = s.mean(0)
        s, tau = s.numpy(), 1.0 / (N + 1)
        for l in range(L):
            for b in range(B):
                st = A.asrkf_get_state(ctx, l, b, N + 8)
                want = (s[l, b] < tau) & (np.arange(N + 1) < N + 1 - 16)
                clear = np.abs(s[l, b] - tau) > 1e-3 * tau
                np.testing.assert_array_equal(st["frozen"][clear], want[clear], err_msg=f"{l} {b}")
                assert 0.2 < want.mean() < 0.8
    finally:
        A.asrkf_destroy(ctx)


@pytest.mark.parametrize("scope", ["layer", "token"])
def test_captured_steps_with_several_verdict_launches(gpu, scope):
    torch = gpu
    import paper_2512_11221_amd as A
    K, V, q = _inputs(torch)
    new = [x[:, :, N].contiguous() for x in (K, V)]
    outs, states = [], []
    for captured in (False, True):
        out = torch.empty((L, B, HQ, D), device="cuda")
        ctx = _context(A, scope, K, V)
        try:
            _step(A, ctx, q, new[0], new[1], out)
            if captured:
                g = torch.cuda.CUDAGraph()
                torch.cuda.synchronize()
                with torch.cuda.graph(g):
                    _step(A, ctx, q, new[0], new[1], out)
            for _ in range(3):
                if captured:
                    g.replay()
                else:
                    _step(A, ctx, q, new[0], new[1], out)
            states.append([A.asrkf_get_state(ctx, l, b, N + 8) for l in range(L) for b in range(B)])
            outs.append(out.cpu())
        finally:
            A.asrkf_destroy(ctx)
    assert torch.equal(outs[0], outs[1])
    for x, y in zip(*states):
        for f in ("unfreeze", "count", "frozen", "active"):
            np.testing.assert_array_equal(x[f], y[f])


def test_one_layers_planes_where_memory_is_short(gpu):
    """With the planes of all layers (2.1 GB) a context would not fit into what is
    left of the device, with one layer's (134 MB) it does, and decodes the same."""
    torch = gpu
    import paper_2512_11221_amd as A
    layers, batch, ctx_len = 16, 4, 1 << 18
    cfg = A.make_config(layers, batch, 32, 8, 128, ctx_len - 1, 16, 2e-3, 0.25, 64, dtype="bf16",
                        relevance="softmax")
    rows = 2 * layers * batch * ctx_len * 2048
    positions = 13 * layers * batch * ctx_len
    g = torch.Generator(device="cuda").manual_seed(29)
    n = 400
    K = torch.randn((n + 1, 8, 128), generator=g, device="cuda", dtype=torch.bfloat16)
    q = torch.randn((batch, 32, 128), generator=g, device="cuda", dtype=torch.bfloat16)
    new = K[n:].expand(batch, 8, 128).contiguous()
    got = []
    for leave in (None, rows + positions + (1 << 30)):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        filler = None
        if leave is not None:
            free = torch.cuda.mem_get_info()[0]
            if free < leave:
                pytest.skip("another program holds the device's memory")
            filler = torch.empty(free - leave, dtype=torch.uint8, device="cuda")
        ctx = None
        try:
            ctx = A.asrkf_init(cfg)
            out = torch.empty((layers, batch, 32, 128), device="cuda")
            for l in range(layers):
                for b in range(batch):
                    A.asrkf_prefill(ctx, l, b, K, K, n)
            for _ in range(3):
                for l in range(layers):
                    A.asrkf_decode_step(ctx, l, q, new, new, out[l])
                A.asrkf_restore(ctx, None, A.NONE)
            got.append((out.cpu(), [A.asrkf_get_state(ctx, l, 1, ctx_len) for l in range(layers)]))
        finally:
            A.asrkf_destroy(ctx)
            del filler
            torch.cuda.empty_cache()
    assert torch.equal(got[0][0], got[1][0])
    for x, y in zip(got[0][1], got[1][1]):
        np.testing.assert_array_equal(x["frozen"], y["frozen"])
        assert 0.1 < x["frozen"].mean() < 0.99
