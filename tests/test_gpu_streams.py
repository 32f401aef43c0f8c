"""The stage hooks follow the work that fills their tensors: with some tens of
milliseconds of work ahead of the inputs' last write on torch's current stream,
the default one or another, a hook returns the same bits as on inputs that are
ready (until then the buffers hold zeros, which every hook accepts)."""
import numpy as np
import pytest

import paper_2608_11249_amd as dl
import workloads as wl
from tests.gpu_common import log, shape

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

V, N, B, T = 4099, 300, 4, 512


def inputs():
    rng = np.random.default_rng(9)
    return dict(logits=wl.random_logits(1, N, V, 3.0), sym=rng.integers(0, V, N).astype(np.int32),
                rank=rng.integers(0, V, N).astype(np.int32),
                H=rng.uniform(0, 8, B * T // 2).astype(np.float32),
                rows=np.arange(0, B * T, 2, dtype=np.int32),
                state=wl.random_state(3, B, T, V, 0.5).astype(np.int32))


HOOKS = {
    "forward_logits": lambda m, x: m.forward_logits(x["state"]),
    "entropy_cdf": lambda m, x: m.entropy_cdf(x["logits"], 24),
    "entropy_cdf_noalloc": lambda m, x: m.entropy_cdf_noalloc(x["logits"], 24),
    "select": lambda m, x: m.select(x["H"], x["rows"], B, T, 0.5, 1, 64),
    "rank_rows": lambda m, x: (m.rank_rows(x["logits"], x["sym"]),),
    "select_rank_rows": lambda m, x: (m.select_rank_rows(x["logits"], x["rank"]),),
}


@pytest.mark.parametrize("side", [False, True], ids=["default", "side"])
@pytest.mark.parametrize("hook", HOOKS)
def test_hooks_wait_for_their_inputs(hook, side):
    ready = {k: torch.from_numpy(a).cuda() for k, a in inputs().items()}
    late = {k: torch.zeros_like(a) for k, a in ready.items()}
    busy = torch.eye(4096, device="cuda")
    out = torch.empty_like(busy)
    torch.mm(busy, busy, out=out)
    with dl.Model(shape(vocab=V, n_layers=1), max_chunk=T, max_batch=B) as m:
        torch.cuda.synchronize()
        want = [t.cpu() for t in HOOKS[hook](m, ready)]
        torch.cuda.synchronize()
        with torch.cuda.stream(torch.cuda.Stream() if side else torch.cuda.default_stream()):
            log("streams", hook, side)
            for _ in range(30):
                torch.mm(busy, busy, out=out)
            for k in late:
                late[k].copy_(ready[k])
            got = HOOKS[hook](m, late)
            torch.cuda.synchronize()
        assert all(torch.equal(a, b.cpu()) for a, b in zip(want, got))
        # calls without tensors afterwards leave the default stream, hooks come back to it
        toks = wl.markov1_tokens(64, V, 1).astype(np.int32)
        scores = m.context_scores(toks)
        again = HOOKS[hook](m, ready)
        assert all(torch.equal(a, b.cpu()) for a, b in zip(want, again))
        assert np.array_equal(scores, m.context_scores(toks))
        m.set_stream(dl.DEFAULT_STREAM)
        assert np.array_equal(scores, m.context_scores(toks))
