"""The prefill's edges at batches wide enough that consecutive positions share a
wavefront and walk the union of their selections, and that queries are listed and
scored again (narrow calls take neither path): the first two sequences against the
oracle at every position, and values that are not finite."""

import numpy as np
import pytest
import torch

import gpu_harness as H
import spla_inputs as si
import test_gpu_prefill as P
import test_gpu_prefill_groups as G
from paper_2601_22379_amd import spla

pytestmark = pytest.mark.gpu

CASES = {n: (spec, {}, T) for n, (spec, T) in G.CASES.items()}
CASES["two_segments"] = (CASES["two_segments"][0], {}, 60)
CASES.update((n, c) for n, c in P.CASES.items() if c[0].get("dtype") != "f32")
base = dict(batch=2, n_q_heads=8, n_kv_heads=2, head_dim=128, block_size=64, top_k=6,
            lengths=[900, 2000], capacity=2112, kind="block_offsets")
FLAGS = {spla.FLAG_NO_RLA: dict(no_rla=True), spla.FLAG_FIRST_ORDER: dict(first_order=True),
         spla.FLAG_RLA_NORMALIZE: dict(rla_normalize=True)}
for f in FLAGS:
    CASES[f"flags{f}"] = (base, dict(flags=f), 20)
CASES["capacity"] = (dict(base, lengths=[1000, 500], capacity=1024, kind="iid"), {}, 40)


def widened(spec, T, kw):
    """spec with its sequences repeated until a call of T positions passes 16384 steps
    of one position each, and its column tiles times statistics tiles pass 512."""
    bh, g = spec["batch"] * spec["n_kv_heads"], spec["n_q_heads"] // spec["n_kv_heads"]
    steps = bh * T * spec["top_k"] * (spec["block_size"] // 32)
    units = spec["capacity"] // kw.get("sel_stride", spec["block_size"])
    n_ct = -(-T // (16 // g))
    n = max(16384 // steps, 512 // (n_ct * -(-units // 64) * bh)) + 1
    return dict(spec, batch=spec["batch"] * n, lengths=list(spec["lengths"]) * n)


@pytest.mark.parametrize("name", list(CASES))
def test_wide_batches_match_the_oracle(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    spec, kw, T = CASES[name]
    w = si.custom(name, code=440 + list(CASES).index(name), **widened(spec, T, kw))
    H.log(f"case {name} T={T} batch={w.batch}")
    cache = spla.SplaCache(H.config_of(w, **kw), dev)
    H.fill_cache(w, cache, lengths=list(w.lengths), device=dev)
    out, sel, q, gamma = P.run_prefill(w, cache, T, dev)
    lens = list(w.lengths)
    assert cache.seq_lens.cpu().tolist() == [min(L + T, w.capacity) for L in lens]
    p = H.params_of(w, window=kw.get("sel_window"), stride=kw.get("sel_stride"),
                    **FLAGS.get(kw.get("flags"), {}))
    at = sorted({t * (T - 1) // 23 for t in range(24)})
    for t in at:
        for b in range(min(2, w.batch)):
            L = min(lens[b] + t + 1, w.capacity)
            for h in range(w.n_kv_heads):
                H.check_kv_head(w, b, h, out[t, b], sel[t, b, h], q[t, b], gamma, p, L=L)


@pytest.mark.parametrize("flags", [0, spla.FLAG_NO_RLA])
def test_values_not_finite_stay_with_their_queries(flags):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    w = si.custom("infwide", 11, 16, 4, 128, 64, 6, [1000] * 11, kind="block_offsets", code=470,
                  capacity=1088)
    kn, vn, q = P.chunk_inputs(w, 33, list(w.lengths))
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
    assert not torch.isfinite(outs[1][21:, :, :, 5]).any()
