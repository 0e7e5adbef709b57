"""Prefills of several chunks, and of more queries than one selection per workgroup,
against appending the rows up to a position and decoding there: selections are the
same, outputs agree to bf16, and the cache ends with the state, statistics and
lengths of one append.

The shapes take three chunks of 1024 positions at most (700 each), or more queries
per compute unit than the selection starts workgroups (32, or 8 with windows), so
that a workgroup selects several, some of them with every block."""

import numpy as np
import pytest
import torch

import gpu_harness as H
import spla_inputs as si
from paper_2601_22379_amd import spla

pytestmark = pytest.mark.gpu

CASES = {
    # lengths that start inside a block; the second sequence starts empty, the last
    # one fills up within the third chunk
    "three_chunks": (dict(batch=3, n_q_heads=8, n_kv_heads=2, head_dim=128, block_size=64, top_k=9,
                          lengths=[130, 0, 1177], capacity=3200, kind="block_offsets"),
                     2100, {}, False),
    "three_chunks_paged": (dict(batch=2, n_q_heads=10, n_kv_heads=2, head_dim=128, block_size=32,
                                top_k=12, lengths=[77, 1300], capacity=3360,
                                kind="pareto_planted"), 2100, {}, True),
    "three_chunks_windows": (dict(batch=2, n_q_heads=4, n_kv_heads=2, head_dim=64, block_size=64,
                                  top_k=8, lengths=[45, 900], capacity=2944, kind="drift"),
                             2100, dict(sel_window=32, sel_stride=16), False),
    "one_head": (dict(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=128, block_size=128, top_k=6,
                      lengths=[1001], capacity=4096, kind="iid"), 2100, {}, False),
    # 12800 queries; the lengths pass top_k blocks within the call
    "many_queries": (dict(batch=16, n_q_heads=16, n_kv_heads=8, head_dim=64, block_size=32,
                          top_k=7, lengths=[120 + 13 * i for i in range(16)], capacity=16384,
                          kind="iid"), 100, {}, False),
    "many_queries_windows": (dict(batch=8, n_q_heads=16, n_kv_heads=8, head_dim=64, block_size=32,
                                  top_k=7, lengths=[120 + 26 * i for i in range(8)], capacity=4096,
                                  kind="block_offsets"), 100,
                             dict(sel_window=16, sel_stride=8), False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_as_appending_and_decoding(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    spec, T, kw, paged = CASES[name]
    w = si.custom(name, code=330 + list(CASES).index(name), **spec)
    nb = w.capacity // w.block_size
    pages, tab = 0, None
    if paged:
        pages = w.batch * nb + 9
        tab = np.random.default_rng(5).permutation(pages)[:w.batch * nb]
        tab = torch.from_numpy(tab.reshape(w.batch, nb).astype(np.int32)).to(dev)
    cfg = spla.make_config(w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim, w.block_size, w.top_k,
                           w.capacity, w.dtype, n_sink=w.n_sink, n_local=w.n_local,
                           kv_pages=pages, **kw)
    K, V, _ = si.gen_kv_slab(w, 0, max(w.lengths) + T, lengths=[L + T for L in w.lengths])
    n = torch.tensor(w.lengths, dtype=torch.int32, device=dev)
    K, V = H.to_dev(K, w, dev), H.to_dev(V, w, dev)
    new = [torch.stack([x[b, :, L:L + T] for b, L in enumerate(w.lengths)]) for x in (K, V)]
    top = max(w.lengths)
    caches = []
    for _ in range(2):
        c = spla.SplaCache(cfg, dev, block_table=tab)
        c.append(K[:, :, :top].contiguous(), V[:, :, :top].contiguous(), n)
        caches.append(c)
    a, b = caches
    q = torch.randn((T, w.batch, w.n_q_heads, w.head_dim),
                    generator=torch.Generator().manual_seed(6)).bfloat16().to(dev)
    gamma = torch.from_numpy(si.gen_gamma(w)).to(dev)
    out, sel = a.prefill(*(x.permute(2, 0, 1, 3).contiguous() for x in new), q, gamma)

    start = [x.clone() for x in (b.stats, b.state, b.norm, b.seq_lens)]
    edges = [0, 1, 2, 698, 699, 700, 701, 702, 1398, 1399, 1400, 1401, 1402, T - 2, T - 1]
    rng = np.random.default_rng(7)
    at = sorted({t for t in edges if t < T} | set(rng.integers(0, T, 60 if T > 100 else 0).tolist())
                | set(range(T if T <= 100 else 0)))
    assert at[-1] == T - 1
    for t in at:
        for x, x0 in zip((b.stats, b.state, b.norm, b.seq_lens), start):
            x.copy_(x0)
        b.append(*(x[:, :, :t + 1].contiguous() for x in new))
        o, s = b.decode(q[t], gamma)
        assert torch.equal(s, sel[t]), (t, int((s != sel[t]).any(-1).sum()))
        err = (out[t].float() - o.float()).abs().amax(-1) / o.float().abs().amax(-1)
        assert err.max() <= H.TOL["bf16"], (t, err.max())
    torch.cuda.synchronize()
    # the last position's append is the whole call's
    assert torch.equal(a.seq_lens, b.seq_lens)
    assert a.seq_lens.tolist() == [min(L + T, w.capacity) for L in w.lengths]
    full = any(L + T > w.capacity for L in w.lengths)
    assert a.device_errors() == (spla.DEVERR_CAPACITY if full else 0)
    if not paged:
        assert torch.equal(a.k, b.k) and torch.equal(a.v, b.v)
    for x, y, rel, tol in ((a.stats, b.stats, 2e-5, 1e-5), (a.state, b.state, 2e-4, 2e-4),
                           (a.norm, b.norm, 2e-5, 1e-5)):
        assert torch.allclose(x, y, rtol=rel, atol=tol), (x - y).abs().max()
