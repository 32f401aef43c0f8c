"""Attention-rollout scores at the edges of their kernels: lengths around the
64-key map tiles, the 16- and 32-row rollout blocks (more than 1024 positions
take 32) and the 256-column ones, odd head counts, every head dim, against the
fp64 oracle.  A score is a sum of T / 2 products of probabilities through the
layers: fp32 keeps it within 1e-4 of the largest, the bf16 model within 3e-2
(its scores' probabilities come from bf16 Q and K)."""
import numpy as np
import pytest

import paper_2608_11249_amd as dl
import workloads as wl
from oracle import context as OX
from oracle import weights as OW
from tests.gpu_common import log, shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H,dh,Ts", [
    ("f32", 3, 16, (1, 2, 17, 65)), ("f32", 1, 32, (63, 257)), ("f32", 3, 64, (64, 130)),
    ("f32", 1, 128, (33,)), ("bf16", 2, 64, (1, 15, 64, 65, 300)), ("bf16", 3, 128, (31, 129)),
    ("bf16", 2, 64, (1025,)), ("bf16", 1, 128, (200,))])
def test_scores_against_the_oracle(dtype, H, dh, Ts):
    sh = shape(d_model=H * dh, n_heads=H, d_ffn=128, vocab=300, dtype=dtype, n_layers=2)
    with dl.Model(sh, max_chunk=max(Ts)) as m:
        for T in Ts:  # ascending: the buffers of a shorter chunk are replaced
            log("context scores", dtype, H, dh, T)
            toks = wl.markov1_tokens(T, sh.vocab, T).astype(np.int32)
            got = m.context_scores(toks).astype(np.float64)
            ref = OX.context_scores(sh, OW.Weights(sh), toks)
            tol = 1e-4 if dtype == "f32" else 3e-2
            assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref)) + 1e-6
            assert np.array_equal(got, m.context_scores(toks))


@pytest.mark.parametrize("dtype,H,dh", [("f32", 3, 16), ("f32", 1, 128), ("bf16", 2, 64), ("bf16", 1, 128)])
def test_shorter_chunk_after_a_longer_one(dtype, H, dh):
    """The buffers of a longer chunk serve a shorter one at its own pitch (an
    input's last chunk): the same bits as on a fresh model, and as the oracle's."""
    sh = shape(d_model=H * dh, n_heads=H, d_ffn=128, vocab=300, dtype=dtype, n_layers=2)
    with dl.Model(sh, max_chunk=700) as used:
        for T in (700, 300, 65, 64, 17, 1, 333):
            log("context scores, shorter", dtype, H, dh, T)
            toks = wl.markov1_tokens(T, sh.vocab, T).astype(np.int32)
            got = used.context_scores(toks)
            with dl.Model(sh, max_chunk=T) as fresh:
                assert np.array_equal(got, fresh.context_scores(toks))
            if T in (17, 65, 333):
                ref = OX.context_scores(sh, OW.Weights(sh), toks)
                tol = 1e-4 if dtype == "f32" else 3e-2
                assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref)) + 1e-6
