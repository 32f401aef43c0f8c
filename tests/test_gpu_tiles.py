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
    # 8B-shaped layer
    "8b": shape(d_model=4096, n_heads=32, d_ffn=12288, vocab=384, n_layers=1, ffn="swiglu", norm="rmsnorm"),
    # LM heads
    "head": shape(d_model=768, n_heads=12, vocab=32768, n_layers=0),
    "head8b": shape(d_model=4096, n_heads=32, vocab=126464, n_layers=0),
}
CASES = [
    ("gelu64", 1, 3), ("gelu64", 63, 5), ("gelu64", 65, 24), ("gelu64", 127, 12), ("gelu64", 129, 31),
    ("gelu64", 389, 33), ("gelu64", 451, 2), ("gelu64", 701, 4), ("gelu64", 897, 6), ("gelu64", 1091, 2),
    ("gelu64", 1367, 3), ("gelu64", 2121, 4), ("gelu64", 2243, 2), ("gelu64", 4121, 3),
    ("swiglu128", 64, 3), ("swiglu128", 128, 9), ("swiglu128", 191, 17), ("swiglu128", 257, 40),
    ("8b", 64, 2), ("8b", 65, 4), ("8b", 129, 4), ("8b", 257, 5), ("8b", 1027, 3), ("8b", 1367, 3),
    ("head", 100, 4), ("head", 130, 2), ("head8b", 65, 4)]


def tiles(sh, M):
    """(epilogue, tile form) of each GEMM of a pass over M rows."""
    d, F = sh.d_model, sh.d_ffn
    glu = sh.ffn == "swiglu"
    gemms = [(sh.vocab, d, "store")]
    if sh.n_layers:
        gemms += [(3 * d, d, "qkv"), (d, d, "residual"), (d, F, "residual"),
                  (2 * F if glu else F, d, "swiglu" if glu else "gelu")]
    out = set()
    for N, K, epi in gemms:
        kind, split = dl.gemm_tiles(M, N, K, epi, d)
        if kind in ("64x64", "128x64"):
            kind += "deep" if split else ""
        elif kind == "4wave":  # columns on 256 x 256 tiles, on 256 x 128, or both
            kind += "256" if split == N else "128" if split == 0 else "split"
        out.add((epi, kind))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("name,T,B", CASES)
def test_chunk_alone_and_in_a_batch_give_the_same_bits(name, T, B):
    import torch
    sh = SHAPES[name]
    log("tiles", name, T, B, sorted(tiles(sh, T)), sorted(tiles(sh, B * T)))
    st = wl.random_state(7, B, T, sh.vocab, 0.5)
    st[:, 0] = sh.mask_id
    dev = torch.from_numpy(st.astype(np.int32)).cuda()
    with dl.Model(sh, max_chunk=T, max_batch=B) as m:
        together, rows = m.forward_logits(dev)
        rows = rows.cpu().numpy()
        assert torch.isfinite(together).all()
        for b in sorted({0, B // 2, B - 1}):
            alone, r1 = m.forward_logits(dev[b:b + 1])
            mine = np.nonzero(rows // T == b)[0]
            assert np.array_equal(r1.cpu().numpy(), rows[mine] - b * T)
            assert torch.equal(alone, together[int(mine[0]):int(mine[-1]) + 1])


def test_cases_reach_every_tile_form_a_model_takes():
    """Every (epilogue, tile form) that the small and the 8B-shaped model take at
    some number of rows is one of the cases' (host only)."""
    rows = [*range(1, 2049), *range(2050, 8192, 7), *range(8192, 65537, 97)]
    taken = set().union(*(tiles(sh, M) for sh in (wl.SMALL, wl.DLM8B) for M in rows))
    reached = set().union(*(tiles(SHAPES[n], M) for n, T, B in CASES for M in (T, T * B)))
    assert taken <= reached, sorted(taken - reached)
    assert len(taken) >= 35


@pytest.mark.parametrize("T", [1, 2, 3, 7, 63, 65, 389, 777, 1023, 1024, 4097, 5461, 8191, 8192])
def test_chunk_of_a_row_by_reciprocal(T):
    """The rotary epilogue's chunk index, (row + 0.5) * (1 / T) in fp32 rounded
    down, is row // T for every row a model can have (host only)."""
    row = np.arange(1 << 20)
    q = (row.astype(np.float32) + np.float32(0.5)) * (np.float32(1.0) / np.float32(T))
    assert np.array_equal(q.astype(np.int64), row // T)
