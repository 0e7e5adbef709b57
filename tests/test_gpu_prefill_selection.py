"""A prefill selects what appending the rows and decoding at each position selects,
also where the block means are large against what tells the blocks apart: the log
masses' partial sums then round at many times the gaps between scores."""

import pytest
import torch

import gpu_harness as H
import spla_inputs as si
from paper_2601_22379_amd import spla

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mean,d,kw", [
    (2.0, 128, {}), (8.0, 128, {}), (16.0, 64, {}), (60.0, 128, {}),
    (16.0, 128, dict(sel_window=32, sel_stride=16)),
    (60.0, 128, dict(flags=spla.FLAG_FIRST_ORDER))])
def test_large_means(mean, d, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    T, hkv, group, L, cap = 512, 8, 2, 65024, 65536
    w = si.custom("means", 1, hkv * group, hkv, d, 32, 24, [L], kind="iid", code=320, capacity=cap)
    g = torch.Generator(device="cuda").manual_seed(int(mean) + d)

    def randn(*shape):
        return torch.randn(shape, generator=g, device=dev)

    common = mean * randn(1, hkv, 1, d)
    K = (common + randn(1, hkv, L, d)).bfloat16()
    V = randn(1, hkv, L, d).bfloat16()
    kn = (common[:, :, 0] + randn(T, 1, hkv, d)).bfloat16()
    vn, q = randn(T, 1, hkv, d).bfloat16(), randn(T, 1, hkv * group, d).bfloat16()
    gamma = torch.ones((hkv * group, d), device=dev)
    a, b = (spla.SplaCache(H.config_of(w, **kw), dev) for _ in range(2))
    for c in (a, b):
        c.append(K, V)
    _, sel = a.prefill(kn, vn, q, gamma)
    start = [x.clone() for x in (b.stats, b.state, b.norm, b.seq_lens)]
    differ = 0
    for t in range(T):
        for x, x0 in zip((b.stats, b.state, b.norm, b.seq_lens), start):
            x.copy_(x0)
        b.append(*(x[:t + 1].permute(1, 2, 0, 3).contiguous() for x in (kn, vn)))
        differ += int((b.decode(q[t], gamma)[1] != sel[t]).any(-1).sum())
    assert differ == 0, f"{differ} of {T * hkv} queries select other blocks than a decode"
