"""spla_step in one launch against the separate launches, step after step: the
outputs, selections and everything the step writes (rows, statistics, state,
lengths) are the same bits. Sequences that start empty, cross a block and a
64-block tile, fill up, or use a small part of a large cache; 8 and 16 sparse
workgroups per head; a paged pool."""

import numpy as np
import pytest
import torch

import gpu_harness as H
import spla_inputs as si
from paper_2601_22379_amd import spla

pytestmark = pytest.mark.gpu

CASES = {
    # 8 sparse workgroups per head; 64-block tiles end at token 4096
    "g4_k16": dict(batch=4, n_q_heads=8, n_kv_heads=2, head_dim=128, block_size=64, top_k=16,
                   lengths=[4093, 0, 700, 16381], capacity=16384, kind="block_offsets"),
    # 16 workgroups per head, one live tile of many
    "g5_k32": dict(batch=2, n_q_heads=10, n_kv_heads=2, head_dim=128, block_size=64, top_k=32,
                   lengths=[62, 2301], capacity=65536, kind="iid"),
    "g1_B128": dict(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=128, block_size=128, top_k=8,
                    lengths=[1278], capacity=2048, kind="drift"),
}


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_one_launch_equals_the_separate_ones(name, paged):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    w = si.custom(name, code=270 + list(CASES).index(name), **CASES[name])
    nb = w.capacity // w.block_size
    pages, tab = 0, None
    if paged:
        pages = w.batch * nb + 5
        tab = np.random.default_rng(1).permutation(pages)[:w.batch * nb]
        tab = torch.from_numpy(tab.reshape(w.batch, nb).astype(np.int32)).to(dev)
    caches = []
    for flags in (0, spla.FLAG_SEPARATE_KERNELS):
        cfg = spla.make_config(w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim, w.block_size,
                               w.top_k, w.capacity, w.dtype, flags=flags, kv_pages=pages)
        c = spla.SplaCache(cfg, dev, block_table=tab)
        H.fill_cache(w, c, lengths=list(w.lengths), device=dev)
        caches.append(c)
    gamma = torch.from_numpy(si.gen_gamma(w)).to(dev)
    rng = np.random.default_rng(2)
    for step in range(6):
        kn, vn = (H.to_dev(rng.standard_normal((w.batch, w.n_kv_heads, w.head_dim)), w, dev)
                  for _ in range(2))
        q = H.to_dev(si.gen_q_batch(w, step), w, dev)
        got = [c.step(kn, vn, q, gamma) for c in caches]
        torch.cuda.synchronize()
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
        for x in ("k", "v", "stats", "state", "norm", "seq_lens"):
            assert torch.equal(getattr(caches[0], x), getattr(caches[1], x)), (step, x)
    assert caches[0].seq_lens.cpu().tolist() == [min(L + 6, w.capacity) for L in w.lengths]
    full = any(L + 6 > w.capacity for L in w.lengths)
    for c in caches:
        assert c.device_errors() == (spla.DEVERR_CAPACITY if full else 0)
