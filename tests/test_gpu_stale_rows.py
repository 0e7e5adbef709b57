"""What the key and value buffers hold past a sequence's length touches no bit of
a result: the same calls on caches whose buffers held zeros, keys whose
exponentials overflow, and NaN before the rows came."""

import pytest
import torch

import gpu_harness as H
import spla_inputs as si
from paper_2601_22379_amd import spla

pytestmark = pytest.mark.gpu

CASES = {
    # every length ends inside a 32-token step; one launch, separate launches, d = 64
    "one_launch": dict(batch=8, n_q_heads=32, n_kv_heads=8, head_dim=128, block_size=64, top_k=8,
                       lengths=[1001, 900, 777, 1203, 650, 1111, 1290, 1005], capacity=1344,
                       kind="block_offsets"),
    "separate": dict(batch=4, n_q_heads=64, n_kv_heads=8, head_dim=128, block_size=64, top_k=8,
                     lengths=[1001, 777, 1203, 650], capacity=1344, kind="block_offsets"),
    "d64": dict(batch=8, n_q_heads=32, n_kv_heads=8, head_dim=64, block_size=32, top_k=8,
                lengths=[1001, 900, 777, 1203, 650, 1111, 1290, 1005], capacity=1344, kind="iid"),
}


def both(name, call):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    w = si.custom(name, code=290 + list(CASES).index(name), **CASES[name])
    got = []
    for stale in (0.0, 100.0, float("nan")):
        cache = spla.SplaCache(H.config_of(w), dev)
        cache.k.fill_(stale)
        cache.v.fill_(stale)
        H.fill_cache(w, cache, lengths=list(w.lengths), device=dev)
        got.append([t.clone() for t in call(w, cache, dev)])
        torch.cuda.synchronize()
    for other in got[1:]:
        for x, y in zip(got[0], other):
            assert torch.equal(x, y), (x.float() - y.float()).abs().max()


@pytest.mark.parametrize("name", list(CASES))
def test_decode_and_step(name):
    def call(w, cache, dev):
        q, gamma = H.to_dev(si.gen_q_batch(w), w, dev), torch.from_numpy(si.gen_gamma(w)).to(dev)
        g = torch.Generator().manual_seed(3)
        rows = [torch.randn((w.batch, w.n_kv_heads, w.head_dim), generator=g).to(dev, q.dtype)
                for _ in range(2)]
        return (*cache.decode(q, gamma), *cache.step(*rows, q, gamma), cache.state, cache.stats)

    both(name, call)


# 3 positions: the last step holds rows of the prefix, which carry linear weights; 41:
# consecutive positions share a wavefront
@pytest.mark.parametrize("T", [3, 41])
@pytest.mark.parametrize("name", list(CASES))
def test_prefill(name, T):
    def call(w, cache, dev):
        q = torch.cat([H.to_dev(si.gen_q_batch(w, t), w, dev)[None] for t in range(T)])
        g = torch.Generator().manual_seed(4)
        rows = [torch.randn((T, w.batch, w.n_kv_heads, w.head_dim), generator=g).to(dev, q.dtype)
                for _ in range(2)]
        return (*cache.prefill(*rows, q, torch.from_numpy(si.gen_gamma(w)).to(dev)), cache.state,
                cache.norm, cache.stats)

    both(name, call)
