"""The fp32 model's kernels (MFMA attention and GEMM) against the fp64 oracle,
at head dims, widths and chunk lengths around their tiles: 64-key attention
tiles, 32 x 64 GEMM tiles with 64-deep k stages, and the widths whose rotary
step is fused into the QKV GEMM (d % 64 == 0, head dim dividing 64) or not."""
import numpy as np
import pytest

import paper_2608_11249_amd as dl
import workloads as wl
from oracle import model as OM
from oracle import weights as OW
from tests.gpu_common import log, rel_err_rows, shape

pytestmark = pytest.mark.gpu

# fp32 rounding (2^-24) through two layers of sums of up to 128 terms, with the
# same margin as the tiny workload's logits
TOL = 1e-5


@pytest.mark.parametrize("kw", [
    dict(d_model=64, n_heads=1, d_ffn=96),                                    # dh 64, fused
    dict(d_model=128, n_heads=8, d_ffn=80),                                   # dh 16, fused; K = 80
    dict(d_model=128, n_heads=1, d_ffn=64, norm="rmsnorm"),                   # dh 128, rotary apart
    dict(d_model=80, n_heads=5, d_ffn=48, ffn="swiglu", norm="rmsnorm"),      # width no multiple of 64
    dict(d_model=96, n_heads=3, d_ffn=112, vocab=67),
], ids=lambda k: f"d{k['d_model']}h{k['n_heads']}")
@pytest.mark.parametrize("B,T", [(1, 1), (2, 17), (1, 63), (3, 64), (2, 65), (1, 130)])
def test_f32_logits_against_oracle(kw, B, T):
    import torch
    sh = shape(dtype="f32", **kw)
    log("f32", kw, B, T)
    st = wl.random_state(5, B, T, sh.vocab, 0.6)
    st[:, 0] = sh.mask_id
    W = OW.Weights(sh)
    with dl.Model(sh, max_chunk=T, max_batch=B) as m:
        lg, rows = m.forward_logits(torch.from_numpy(st.astype(np.int32)).cuda())
        lg, rows = lg.cpu().numpy(), rows.cpu().numpy()
        alone, _ = m.forward_logits(torch.from_numpy(st[-1:].astype(np.int32)).cuda())
    ref = [OM.logits(sh, W, st[b]) for b in range(B)]
    assert np.array_equal(rows, np.concatenate([b * T + ref[b][1] for b in range(B)]))
    assert rel_err_rows(lg, np.concatenate([r[0] for r in ref])) <= TOL
    assert np.array_equal(alone.cpu().numpy(), lg[len(lg) - len(ref[-1][1]):])
