"""The coding stages' kernels at the sizes where their forms change: selection by
256 or 1024 threads, CDFs by rows or in segments, row statistics by one block or
spread over the chip, rank selection by bins or by radix, compaction around its
64-position words and 65536-position spans.
Whole numbers are compared exactly with NumPy."""
import numpy as np
import pytest

import paper_2608_11249_amd as dl
import workloads as wl
from oracle import schedule as OS
from tests.gpu_common import log, shape

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def handle(vocab=256, max_batch=1):
    return dl.Model(shape(vocab=vocab, n_layers=0), max_chunk=1, max_batch=max_batch)


@pytest.mark.parametrize("T,B,frac", [(1, 3, 1.0), (255, 2, 1.0), (257, 3, 0.9), (2048, 4, 1.0),
                                      (2049, 2, 1.0), (8192, 2, 1.0), (8192, 8, 0.2)])
@pytest.mark.parametrize("tau,m_min,m_max", [(float("-inf"), 8, 8), (0.5, 1, 64), (9.0, 1, 1024)])
def test_select_sizes(T, B, frac, tau, m_min, m_max):
    log("select", T, B, frac, tau)
    rng = np.random.default_rng(T + B)
    rows = np.sort(rng.choice(B * T, max(1, int(B * T * frac)), replace=False)).astype(np.int32)
    H = np.round(rng.uniform(0, 8, len(rows)), 2).astype(np.float32)  # many ties
    H[:: 7] = -0.0
    with handle(max_batch=B) as m:
        sp, sr, ns = (t.cpu().numpy() for t in m.select(torch.from_numpy(H).cuda(), torch.from_numpy(rows).cuda(),
                                                        B, T, tau, m_min, m_max))
    for b in range(B):
        seg = np.nonzero((rows >= b * T) & (rows < (b + 1) * T))[0]
        h = H[seg]
        n = min(len(seg), max(m_min, min(m_max, int((h <= tau).sum()))))
        # order of the 32-bit keys: -0 before +0
        key = h.view(np.uint32)
        key = np.where(key >> 31, ~key, key | 0x80000000)
        want = np.sort(np.lexsort((np.arange(len(seg)), key))[:n])
        assert ns[b] == n
        assert np.array_equal(sp[b, :n], rows[seg[want]] - b * T)
        assert np.array_equal(sr[b, :n], seg[want])


@pytest.mark.parametrize("V,n", [(7, 5), (1024, 3), (1025, 2), (4096, 130), (4097, 2), (4097, 128),
                                 (16385, 129), (32768, 128), (32769, 128), (50257, 3), (8191, 300)])
@pytest.mark.parametrize("P,scale", [(17, 9.0), (24, 0.5), (31, 2.0)])
def test_cdf_rows_exact_from_g(V, n, P, scale):
    log("cdf", V, n, P, scale)
    lg = torch.from_numpy(wl.random_logits(V + P, n, V, scale)).cuda()
    lg[0, V // 2] = float("-inf")
    lg[n - 1] = 1.25                                     # all equal: every g is 2^24
    with handle(V) as m:
        H, mx, g, cdf = (t.cpu().numpy() for t in m.entropy_cdf(lg, P))
        H2, mx2, g2, cdf2 = (t.cpu().numpy() for t in m.entropy_cdf_noalloc(lg, P))
        only_H = m.entropy_cdf(lg, P, want_cdf=False)[0].cpu().numpy()
    for x, y in ((H, H2), (mx, mx2), (g, g2), (cdf, cdf2), (H, only_H)):
        assert np.array_equal(x, y)                      # either form of the statistics
    ref = lg.cpu().numpy()
    assert np.array_equal(mx, ref.max(1))
    p = np.exp(ref.astype(np.float64) - mx[:, None])
    assert np.abs(g - np.floor(p * 2.0 ** 24)).max() <= 2  # one expf and product: 2 ulp of 2^24
    p /= p.sum(1, keepdims=True)
    with np.errstate(divide="ignore", invalid="ignore"):
        h64 = -np.where(p > 0, p * np.log2(p), 0.0).sum(1)
    # logs and sums of V terms in fp32, relative to log2 V bits
    assert np.abs(H - h64).max() <= 1e-5 * max(1.0, np.log2(V))
    for i in sorted({0, n // 2, n - 1}):
        gi = g[i].astype(object)
        f = 1 + gi * (2 ** P - V) // int(gi.sum())
        f[int(np.argmax(g[i]))] += 2 ** P - int(f.sum())
        want = np.concatenate([[0], np.cumsum(f)]).astype(np.int64)
        assert np.array_equal(cdf[i].view(np.uint32).astype(np.int64), want)


@pytest.mark.parametrize("V", [129, 257, 300, 8193, 8320])
def test_a_nan_makes_its_rows_entropy_nan(V):
    """Wherever the NaN is -- alone in the last group of 128 columns, all of a
    group, among -inf -- and in every form of the statistics; a group of -inf
    alone carries nothing."""
    log("nan rows", V)
    g0 = (V - 1) // 128 * 128                            # the last group
    n = 6
    lg = wl.random_logits(V, n, V, 2.0)
    lg[1, g0:] = np.nan
    lg[2, :128] = np.nan
    lg[3, g0:] = -np.inf
    lg[3, V - 1] = np.nan
    lg[4, g0:] = -np.inf
    lg[4, 0] = 1.0
    dev = torch.from_numpy(lg).cuda()
    with handle(V) as m:
        forms = [m.entropy_cdf(dev, 24, want_cdf=c)[0].cpu().numpy() for c in (True, False)]
        forms.append(m.entropy_cdf_noalloc(dev, 24)[0].cpu().numpy())
        many = m.entropy_cdf(dev.repeat(50, 1), 24)[0].cpu().numpy()
    for H in forms:
        assert np.array_equal(H, many[:n], equal_nan=True)
        assert np.isnan(H[1:4]).all() and np.isfinite(H[[0, 4, 5]]).all()


@pytest.mark.parametrize("V", [2, 63, 1025, 32768, 40000])
def test_rank_rows_forms(V):
    log("rank", V)
    rng = np.random.default_rng(V)
    n = 15
    lg = rng.normal(0, 3, (n, V)).astype(np.float32)
    lg[1] = 0.5                                          # one value: no bins
    lg[2] = np.round(lg[2])                              # ties, more than fit the candidate list
    lg[3, V // 2] = -np.inf
    lg[4, 0] = np.inf
    lg[5, : V // 2] = 0.0
    lg[5, V // 2:] = -0.0                                # equal to +0
    lg[6] = 3.0e38 * np.sign(lg[6])                      # the range overflows
    lg[7, 0] = 1e4                                       # all others in one bin
    lg[8] *= 1e-42                                       # denormals
    lg[9, V - 1] = -1e4                                  # the same from below
    lg[10, ::2] = -np.inf
    lg[11] = np.exp(4 * lg[11])                          # over 60 octaves
    lg[12] = np.round(lg[12])
    lg[12, 0] = 1e6                                      # few values, all in one bin
    lg[13] = -np.inf
    lg[14, V // 3:] = 1.0 + 2.0 ** -20 * (np.arange(V - V // 3) % 7)  # apart in the last key bits
    lg[14, 0] = 1e6
    order = np.argsort(-(lg + 0.0).astype(np.float64), axis=1, kind="stable")
    with handle(V) as m:
        dev = torch.from_numpy(lg).cuda()
        for r in sorted({0, 1, V // 3, V // 2, V - 2, V - 1}):
            rank = torch.full((n,), r, dtype=torch.int32, device="cuda")
            sym = m.select_rank_rows(dev, rank)
            assert np.array_equal(sym.cpu().numpy(), order[:, r]), r
            assert np.array_equal(m.rank_rows(dev, sym).cpu().numpy(), rank.cpu().numpy()), r
        for bad in (-1, V):
            with pytest.raises(dl.DlmcError) as e:
                m.select_rank_rows(dev, torch.full((n,), bad, dtype=torch.int32, device="cuda"))
            assert e.value.code == -1


@pytest.mark.parametrize("n,bad", [(1, 0), (9, 8), (1024, 0), (1025, 1024), (5000, 4321)])
def test_a_rank_outside_the_alphabet_leaves_the_symbols_alone(n, bad):
    log("bad rank", n, bad)
    V = 67
    lg = torch.from_numpy(wl.random_logits(n, n, V, 2.0)).cuda()
    good = torch.arange(n, dtype=torch.int32, device="cuda") % V
    call = dl.lib().dlmc_select_rank_rows
    with handle(V) as m:
        want = m.select_rank_rows(lg, good)
        for wrong in (-1, V, 2 ** 31 - 1):
            rank = good.clone()
            rank[bad] = wrong
            sym = torch.full_like(rank, -7)
            torch.cuda.synchronize()
            assert call(m.handle, lg.data_ptr(), n, rank.data_ptr(), sym.data_ptr()) == -1
            assert (sym == -7).all()
        sym = good.clone()                               # in place
        torch.cuda.synchronize()
        assert call(m.handle, lg.data_ptr(), n, sym.data_ptr(), sym.data_ptr()) == 0
        assert torch.equal(sym, want)


@pytest.mark.parametrize("B,T", [(1, 1), (1, 63), (3, 65), (5, 1000), (64, 1024), (40, 1700), (9, 8192)])
def test_compaction_spans(B, T):
    """Masked rows of a forward pass, over one and several 65536-position spans."""
    log("compact", B, T)
    sh = shape(vocab=3, n_layers=0)
    st = np.random.default_rng(B).choice([0, 1, 2, 3], (B, T), p=[0.3, 0.3, 0.3, 0.1])
    st[0] = 0                                            # nothing masked
    st[-1, -1] = 3
    if B > 2:
        st[1] = 3                                        # all masked
    with dl.Model(sh, max_chunk=T, max_batch=B) as m:
        _, rows = m.forward_logits(torch.from_numpy(st.astype(np.int32)).cuda())
    assert np.array_equal(rows.cpu().numpy(), np.nonzero(st.reshape(-1) == 3)[0])


def test_order_of_tied_entropies_matches_the_oracle():
    H = np.array([0.5, 0.25, 0.5, 0.25, 0.25], np.float32)
    rows = np.arange(5, dtype=np.int32)
    with handle() as m:
        sp, _, ns = m.select(torch.from_numpy(H).cuda(), torch.from_numpy(rows).cuda(), 1, 5,
                             float("-inf"), 4, 4)
    ref = OS.select(H.astype(np.float64), rows, float("-inf"), 4, 4)
    assert np.array_equal(sp.cpu().numpy()[0, : int(ns[0])], ref)
