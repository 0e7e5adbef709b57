"""Prefill where blocks repeat, so that block scores tie at the cutoff and every
query's masses are taken again with the decode's sums: the selections are the
decode's for every count of heads that a tile's 16 columns hold, with and without
strided windows, and such a call costs a small multiple of one without ties."""

import numpy as np
import pytest
import torch

import gpu_harness as H
import spla_inputs as si
from paper_2601_22379_amd import spla
from test_gpu_prefill import chunk_inputs

pytestmark = pytest.mark.gpu


def filled(w, dev, repeat, **kw):
    """A cache in which block i holds block i % repeat's keys (0: its own)."""
    K, V, n = si.gen_kv_slab(w, 0, max(w.lengths))
    if repeat:
        K = K[:, :, np.arange(max(w.lengths)) % (repeat * w.block_size)]
    cache = spla.SplaCache(H.config_of(w, **kw), dev)
    cache.append(H.to_dev(K, w, dev), H.to_dev(V, w, dev), torch.from_numpy(n).to(dev))
    return cache


# queries per column tile: 16, 8, 5, 4, 3, 2; more than one tile's worth of each
@pytest.mark.parametrize("group,d,B,kw", [
    (1, 128, 64, {}), (2, 64, 32, {}), (3, 128, 64, {}), (4, 128, 64, {}), (5, 128, 128, {}),
    (8, 128, 64, {}), (4, 128, 64, dict(sel_window=32, sel_stride=16)),
    (8, 64, 64, dict(sel_window=16, sel_stride=16)),
    (2, 128, 64, dict(flags=spla.FLAG_FIRST_ORDER))])
def test_listed_queries_select_as_a_decode(group, d, B, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    # (wide and long enough that the queries are listed rather than scored exactly at once)
    w = si.custom("ties", 6, 2 * group, 2, d, B, 7, [4500, 3000] * 3, kind="iid",
                  code=300 + group, capacity=65536)
    T = 37
    kn, vn, q = chunk_inputs(w, T, list(w.lengths))
    gamma = torch.from_numpy(si.gen_gamma(w)).to(dev)
    kn, vn, q = (H.to_dev(x, w, dev) for x in (kn, vn, q))
    a, b = filled(w, dev, 3, **kw), filled(w, dev, 3, **kw)
    out, sel = a.prefill(kn, vn, q, gamma)
    # position t: the t + 1 rows appended at once (token by token the statistics
    # are rounded to fp32 after each), then a decode
    start = [x.clone() for x in (b.stats, b.state, b.norm, b.seq_lens)]
    steps = []
    for t in range(T):
        for x, x0 in zip((b.stats, b.state, b.norm, b.seq_lens), start):
            x.copy_(x0)
        b.append(*(x[:t + 1].permute(1, 2, 0, 3).contiguous() for x in (kn, vn)))
        steps.append(b.decode(q[t], gamma))
    torch.cuda.synchronize()
    assert torch.equal(sel, torch.stack([s for _, s in steps]))
    got, want = out.float(), torch.stack([o for o, _ in steps]).float()
    assert ((got - want).abs().amax(-1) <= 2e-2 * want.abs().amax(-1)).all()


def test_ties_cost_a_small_multiple():
    """1024 positions at 512 blocks, every query listed: 8 times the call without
    ties when the listed queries went one by one, about 2 times now."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    w = si.custom("tiescost", 1, 32, 8, 128, 64, 16, [32256], kind="iid", code=310,
                  capacity=33280)
    T = 1000
    g = torch.Generator(device="cuda").manual_seed(1)
    kn, vn, q = (torch.randn((T, 1, h, 128), generator=g, device=dev).bfloat16()
                 for h in (8, 8, 32))
    gamma = torch.from_numpy(si.gen_gamma(w)).to(dev)
    took = []
    for repeat in (0, 4):
        cache = filled(w, dev, repeat)
        n0 = cache.seq_lens.clone()
        best = 1e9
        for _ in range(5):
            cache.seq_lens.copy_(n0)
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            cache.prefill(kn, vn, q, gamma)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        took.append(best)
    H.log(f"prefill without ties {took[0]:.3f} ms, with {took[1]:.3f} ms")
    assert took[1] < 4 * took[0], took
