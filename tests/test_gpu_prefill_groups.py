"""The prefill's group pass, scoring and selection at the edges of their tiles:
group sizes that leave matrix-core columns idle, positions that start inside a
block, chunks that split a group's blocks over workgroups, more blocks than one
pass over the union holds, keys whose exponentials need the shifted form, values
that are not finite, equal block scores; and the workspace query.
"""

import numpy as np
import pytest
import torch

import gpu_harness as H
import spla_inputs as si
from paper_2601_22379_amd import spla
from test_gpu_prefill import check_positions, chunk_inputs, run_prefill

CASES = {
    # 16 positions per wavefront, no forced blocks: the positions' own block may be unselected
    "g1_B32": (dict(batch=1, n_q_heads=2, n_kv_heads=2, head_dim=128, block_size=32, top_k=4,
                    lengths=[45], capacity=160, kind="block_offsets", n_sink=0, n_local=0), 77),
    "g3_d64": (dict(batch=2, n_q_heads=3, n_kv_heads=1, head_dim=64, block_size=64, top_k=5,
                    lengths=[700, 3], capacity=832, kind="drift", n_sink=0, n_local=0), 67),
    "g5": (dict(batch=1, n_q_heads=10, n_kv_heads=2, head_dim=128, block_size=64, top_k=6,
                lengths=[1001], capacity=1152, kind="pareto_planted", n_sink=1, n_local=0), 37),
    "g7_B128": (dict(batch=1, n_q_heads=7, n_kv_heads=1, head_dim=128, block_size=128, top_k=3,
                     lengths=[1279], capacity=1408, kind="iid", n_sink=0, n_local=1), 19),
    # two passes over the union (1063 blocks), one (sequence, KV head): blocks split widely
    "two_segments": (dict(batch=1, n_q_heads=2, n_kv_heads=1, head_dim=64, block_size=32,
                          top_k=40, lengths=[34000], capacity=34048, kind="iid"), 5),
    # exp(k) overflows without the shift by the row maximum
    "large_keys": (dict(batch=1, n_q_heads=4, n_kv_heads=1, head_dim=128, block_size=64, top_k=6,
                        lengths=[777], capacity=896, kind="block_offsets", offset_std=60.0), 20),
}


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    spla.lib()
    return torch.device("cuda:0")


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_group_edges_match_the_oracle(dev, name):
    spec, T = CASES[name]
    w = si.custom(name, code=240 + list(CASES).index(name), **spec)
    cache = spla.SplaCache(H.config_of(w), dev)
    H.fill_cache(w, cache, lengths=list(w.lengths), device=dev)
    out, sel, q, gamma = run_prefill(w, cache, T, dev)
    assert cache.device_errors() == 0
    check_positions(w, out, sel, q, gamma, H.params_of(w), list(w.lengths), T)


@pytest.mark.gpu
@pytest.mark.parametrize("kind,repeat", [("iid", 0), ("pareto_planted", 0), ("iid", 4)])
def test_selection_is_the_decodes(dev, kind, repeat):
    """Every position selects the blocks a decode step there selects, also
    where blocks repeat (repeat: block i holds block i % repeat's keys, so
    whole runs of scores are equal and the lower ids win)."""
    w = si.custom("seldec", 1, 8, 2, 128, 64, 9, [2500], kind=kind, code=250 + repeat,
                  capacity=2624)
    T, L, B = 40, w.lengths[0], w.block_size
    K, V, n = si.gen_kv_slab(w, 0, L)
    if repeat:
        K = K[:, :, np.arange(L) % (repeat * B)]
    kn, vn, q = chunk_inputs(w, T, list(w.lengths))
    gamma = torch.from_numpy(si.gen_gamma(w)).to(dev)
    kn, vn, q = (H.to_dev(x, w, dev) for x in (kn, vn, q))
    sels = []
    for stepwise in (False, True):
        cache = spla.SplaCache(H.config_of(w), dev)
        cache.append(H.to_dev(K, w, dev), H.to_dev(V, w, dev), torch.from_numpy(n).to(dev))
        if stepwise:
            sels.append(torch.stack([cache.step(kn[t], vn[t], q[t], gamma)[1] for t in range(T)]))
        else:
            sels.append(cache.prefill(kn, vn, q, gamma)[1])
    torch.cuda.synchronize()
    assert torch.equal(sels[0], sels[1])


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, spla.FLAG_NO_RLA])
def test_values_not_finite_stay_with_their_queries(dev, flags):
    """An infinite value at position 21 reaches the queries from 21 on and
    leaves the earlier ones of the same wavefront and chunk bit for bit."""
    w = si.custom("inf", 1, 4, 1, 128, 64, 6, [1000], kind="block_offsets", code=260,
                  capacity=1088)
    kn, vn, q = chunk_inputs(w, 33, list(w.lengths))
    gamma = torch.from_numpy(si.gen_gamma(w)).to(dev)
    outs = []
    for bad in (False, True):
        cache = spla.SplaCache(H.config_of(w, flags=flags), dev)
        H.fill_cache(w, cache, device=dev)
        if bad:
            vn[21, :, :, 5] = np.inf
        outs.append(cache.prefill(H.to_dev(kn, w, dev), H.to_dev(vn, w, dev),
                                  H.to_dev(q, w, dev), gamma)[0].float())
    torch.cuda.synchronize()
    assert torch.equal(outs[0][:21], outs[1][:21])
    assert not torch.isfinite(outs[1][21:, 0, :, 5]).any()


@pytest.mark.parametrize("batch,hkv,group,d,B,k,cap", [
    (1, 1, 1, 64, 32, 8, 1 << 20), (4, 8, 4, 128, 64, 32, 131072), (64, 8, 4, 128, 128, 16, 65536),
    (1, 8, 5, 128, 64, 32, 131072), (2, 2, 8, 128, 32, 256, 8192)])
def test_workspace_grows_with_the_positions(batch, hkv, group, d, B, k, cap):
    """A workspace sized for n positions serves every smaller call."""
    cfg = spla.make_config(batch, hkv * group, hkv, d, B, k, cap)
    sizes = [spla.prefill_workspace_bytes(cfg, n, library=spla.host_lib())
             for n in range(0, min(cap, 2100))]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))
