"""A chunk's logits do not depend on what earlier passes of other lengths left in
the workspace (the padding rows of Q, K and V): the same bits on a used model
as on a fresh one, for lengths off the 32-query and 64-key tiles."""
import numpy as np
import pytest

import paper_2608_11249_amd as dl
import workloads as wl
from tests.gpu_common import log, shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H,dh", [("bf16", 2, 64), ("bf16", 1, 128), ("f32", 3, 16), ("f32", 4, 32),
                                        ("f32", 2, 64), ("f32", 1, 128)])
@pytest.mark.parametrize("T", [1, 33, 95, 129, 389])
def test_short_chunk_after_long_ones(dtype, H, dh, T):
    import torch
    # sharpened attention, so that the softmax maxima move between key tiles
    d = H * dh
    sh = shape(d_model=d, n_heads=H, d_ffn=128, vocab=300, dtype=dtype, attn_exp=wl.fan_in_exp(d) - 2)
    log("stale rows", dtype, H, dh, T)
    dev = torch.from_numpy(wl.random_state(3, 1, T, sh.vocab, 1.0).astype(np.int32)).cuda()
    big = torch.from_numpy(wl.random_state(4, 2, 640, sh.vocab, 0.5).astype(np.int32)).cuda()
    with dl.Model(sh, max_chunk=640, max_batch=2) as m:
        fresh = m.forward_logits(dev)[0].cpu().numpy()
        m.forward_logits(big)
        again = m.forward_logits(dev)[0].cpu().numpy()
    assert np.isfinite(fresh).all() and np.array_equal(fresh, again)
