"""Entropy over vocabularies and logits rows that start at any 4-byte boundary
(16-byte loads from the first boundary on, the rest apart), and the counters and
monitors that a waiting call reads back after resets.

Bound: the fp32 entropy of V terms merges log2(V) levels of triples; 1e-5 nats at
V = 128256 was measured for aligned rows, and 5e-5 leaves a factor of five."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11221_amd as A
    A.load()
    return torch


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
@pytest.mark.parametrize("vocab", [1, 2, 3, 4, 5, 7, 63, 1021, 4099, 50257])
def test_any_row_start(gpu, vocab, offset):
    torch = gpu
    import paper_2512_11221_amd as A
    B = 3
    g = torch.Generator(device="cuda").manual_seed(13 * vocab + offset)
    flat = torch.randn(B * vocab + 4, generator=g, device="cuda") * 3.0
    logits = flat[offset:offset + B * vocab].view(B, vocab)
    if vocab > 4:
        logits[1, 0] = -float("inf")          # a probability of 0 among the leading logits
        logits[2, vocab - 1] = -float("inf")  # and the last one
    ctx = A.asrkf_init(A.make_config(1, B, 8, 2, 64, 8, 2, 0.5, 2.0, vocab, dtype="bf16"))
    try:
        q = torch.randn((B, 8, 64), generator=g, device="cuda").to(torch.bfloat16)
        k = torch.randn((B, 2, 64), generator=g, device="cuda").to(torch.bfloat16)
        out = torch.empty((B, 8, 64), device="cuda")
        for rep in range(2):                  # the second time after a reset
            A.asrkf_decode_step(ctx, 0, q, k, k, out)
            A.asrkf_restore(ctx, logits, A.WR)
            for b in range(B):
                x = logits[b].double().cpu().numpy()
                want, pmax = oracle.entropy(x)
                got = A.asrkf_get_seq(ctx, b)
                assert abs(got["entropy"] - want) <= 5e-5 and abs(got["pmax"] - pmax) <= 5e-6
                assert got["level"] == 2 and got["escalation"] == 0
            st = A.asrkf_stats(ctx)
            assert st["step"] == 1 and st["recoveries"][2] == B and st["attended_total"] == B
            A.asrkf_reset(ctx)
            st = A.asrkf_stats(ctx)
            assert st["step"] == 0 and st["recoveries"] == [0, 0, 0, 0] and st["attended_total"] == 0
            assert A.asrkf_get_seq(ctx, 1) == {"entropy": 0.0, "pmax": 0.0, "escalation": 0, "level": 0}
    finally:
        A.asrkf_destroy(ctx)
