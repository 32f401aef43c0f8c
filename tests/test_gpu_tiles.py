"""GEMM tile shapes at their edges: a chunk's logits are the same bits whether it
runs alone (64 x 64, 128 x 64 or deep 128 x 128 tiles of the ring kernel) or
among others (the larger tiles), for row counts around the tile sizes.  The
sums over k have one order in every kernel, so no tolerance is needed; the
values themselves are held against the fp64 oracle elsewhere."""
import numpy as np
import pytest

import paper_2608_11249_amd as dl
import workloads as wl
from tests.gpu_common import log, shape

SHAPES = {
    # small-model layer (K = 768, 3072), head dim 64
    "gelu64": shape(d_model=768, n_heads=12, d_ffn=3072, vocab=384, n_layers=1),
    # head dim 128, SwiGLU with an F that is no multiple of 128
    "swiglu128": shape(d_model=1024, n_heads=8, d_ffn=2112, vocab=384, n_layers=1, ffn="swiglu",
                       norm="rmsnorm"),
}


def layer_tiles(sh, M):
    d, F = sh.d_model, sh.d_ffn
    glu = sh.ffn == "swiglu"
    return {dl.gemm_tiles(M, 3 * d, d, "qkv", d)[0], dl.gemm_tiles(M, d, d, "residual", d)[0],
            dl.gemm_tiles(M, 2 * F if glu else F, d, "swiglu" if glu else "gelu", d)[0],
            dl.gemm_tiles(M, d, F, "residual", d)[0]}


@pytest.mark.gpu
@pytest.mark.parametrize("name,T,B", [
    ("gelu64", 1, 3), ("gelu64", 63, 5), ("gelu64", 65, 24), ("gelu64", 127, 12), ("gelu64", 129, 31),
    ("gelu64", 389, 33), ("swiglu128", 64, 3), ("swiglu128", 128, 9), ("swiglu128", 191, 17),
    ("swiglu128", 257, 40)])
def test_chunk_alone_and_in_a_batch_give_the_same_bits(name, T, B):
    import torch
    sh = SHAPES[name]
    log("tiles", name, T, B, sorted(layer_tiles(sh, T)), sorted(layer_tiles(sh, B * T)))
    st = wl.random_state(7, B, T, sh.vocab, 0.5)
    st[:, 0] = sh.mask_id
    dev = torch.from_numpy(st.astype(np.int32)).cuda()
    with dl.Model(sh, max_chunk=T, max_batch=B) as m:
        together, rows = m.forward_logits(dev)
        together, rows = together.cpu().numpy(), rows.cpu().numpy()
        assert np.isfinite(together).all()
        for b in sorted({0, B // 2, B - 1}):
            alone, r1 = m.forward_logits(dev[b:b + 1])
            mine = rows // T == b
            assert np.array_equal(r1.cpu().numpy(), rows[mine] - b * T)
            assert np.array_equal(alone.cpu().numpy(), together[mine])


def test_few_rows_take_the_ring_tiles():
    """The cases above reach every ring tile shape and the larger ones (host only)."""
    few = set().union(*(layer_tiles(SHAPES[n], T) for n, T in
                        (("gelu64", 63), ("gelu64", 389), ("swiglu128", 191))))
    many = set().union(*(layer_tiles(SHAPES[n], T * B) for n, T, B in
                         (("gelu64", 65, 24), ("gelu64", 389, 33), ("swiglu128", 257, 40))))
    assert "64x64" in few
    assert many - {"64x64"}


@pytest.mark.parametrize("T", [1, 2, 3, 7, 63, 65, 389, 777, 1023, 1024, 4097, 5461, 8191, 8192])
def test_chunk_of_a_row_by_reciprocal(T):
    """The rotary epilogue's chunk index, (row + 0.5) * (1 / T) in fp32 rounded
    down, is row // T for every row a model can have (host only)."""
    row = np.arange(1 << 20)
    q = (row.astype(np.float32) + np.float32(0.5)) * (np.float32(1.0) / np.float32(T))
    assert np.array_equal(q.astype(np.int64), row // T)
