"""The end-of-step rebuild at the sizes where its form changes: up to 8192
positions (two tiles) one launch walks an instance, above that an instance is cut
into segments of 4096 positions and two launches count and write.  Ragged
sequences whose lengths pass a segment's edge during the run, an empty and a
short one beside them; both state scopes, a finite history window, and every
forced recovery level.  Every candidate scores below tau, so thousands of states
change at each step; states and lists must equal the oracle's bit for bit."""
import math

import pytest

from synth import gen
from tests import _harness as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11221_amd as A
    A.load()


def _workload(max_ctx, steps, **kw):
    args = dict(name="rebuild", seed=gen.SEED + 211, n_layers=2, batch=5, n_q_heads=4, n_kv_heads=1,
                head_dim=64, dtype="bf16", prefill=[max_ctx - steps, 4091, 4096, 0, 130], steps=steps,
                window_K=20, tau=math.inf, k_soft=0.5, vocab=64, logit_sigma=1.0, recipe="gauss",
                wr_last_N=4200)
    args.update(kw)
    w = gen.Workload(**args)
    return w.replace(max_ctx=max_ctx)


def _parity(w, modes=None):
    inst = [(l, b) for l in range(w.n_layers) for b in range(w.batch)]
    g, _, stats = H.run_gpu(w, H.Inputs(w), inst, modes=modes)
    o = H.run_oracle(w, H.Inputs(w), inst, modes=modes)
    for k in inst:
        H.compare_instance(g[k], o[k])
    return stats


@pytest.mark.parametrize("history_W", [0, 4])
@pytest.mark.parametrize("scope", ["layer", "token"])
@pytest.mark.parametrize("max_ctx", [8191, 8192])
def test_forced_recovery_on_both_sides_of_the_limit(max_ctx, scope, history_W):
    """8191 is the last max_ctx of the one-launch form (8192 positions), 8192 the
    first of the two-launch form.  Window Reset reaches back past a segment's edge."""
    import paper_2512_11221_amd as A
    w = _workload(max_ctx, 9, scope=scope, history_W=history_W)
    stats = _parity(w, modes={3: A.SR, 5: A.WR, 7: A.FR, 9: A.SR})
    assert stats[-1]["recoveries"] == [0, 2 * w.batch, w.batch, w.batch]


@pytest.mark.parametrize("scope", ["layer", "token"])
def test_edges_of_the_segments(scope):
    """Lengths that reach, end at and pass the edges at 4096 and 8192 positions."""
    w = _workload(12300, 6, scope=scope, prefill=[4090, 4095, 8187, 8192, 12289], batch=5)
    _parity(w)
