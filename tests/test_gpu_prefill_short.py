"""Prefills of a few positions: scored with the decode's sums at once (one 16-column
tile of query rows, a few, or more than that), and attended by one wavefront per
position or per group of positions, whose blocks one, two or many wavefronts share.
Every position selects what a decode there does, and a short prefill costs no more
than the steps it replaces."""

import pytest
import torch

import gpu_harness as H
import spla_inputs as si
from paper_2601_22379_amd import spla
from test_gpu_prefill import chunk_inputs
from test_gpu_prefill_ties import filled

pytestmark = pytest.mark.gpu


# n column tiles of 16 // group positions; positions x k x B / 32 x heads against
# 16384 steps (one position per wavefront up to there)
@pytest.mark.parametrize("batch,hkv,group,d,B,k,T,kw", [
    (2, 2, 4, 128, 64, 7, 1, {}), (2, 2, 4, 128, 64, 7, 4, {}), (2, 2, 4, 128, 64, 7, 5, {}),
    (2, 2, 8, 128, 64, 7, 2, {}), (2, 2, 8, 128, 64, 7, 3, {}), (1, 1, 1, 64, 32, 6, 16, {}),
    (1, 1, 1, 64, 32, 6, 17, {}), (2, 2, 5, 128, 64, 7, 3, {}), (2, 2, 5, 128, 64, 7, 9, {}),
    (2, 2, 3, 64, 64, 7, 5, dict(flags=spla.FLAG_FIRST_ORDER)),
    (2, 2, 4, 128, 64, 7, 33, dict(sel_window=32, sel_stride=16)),
    # no local block: the block in progress is walked though it is not selected
    (2, 2, 4, 128, 64, 7, 6, dict(n_local=0)), (2, 2, 4, 128, 64, 7, 3, dict(n_local=0)),
    (1, 1, 2, 128, 64, 256, 8, {}),                                  # the longest selection
    (8, 8, 4, 128, 128, 32, 3, {}), (8, 8, 4, 128, 128, 32, 2, {}),  # groups; one each
    (8, 8, 2, 64, 32, 64, 6, {}), (16, 8, 4, 64, 64, 24, 21, {})])
def test_positions_select_as_a_decode(batch, hkv, group, d, B, k, T, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    kw = dict(kw)
    local = kw.pop("n_local", 4)
    cap = (k + 24) * B
    lens = [cap - 2 * B - 3 - 7 * b for b in range(batch)]
    w = si.custom("short", batch, hkv * group, hkv, d, B, k, lens, kind="iid", code=400 + group,
                  capacity=cap, n_local=local)
    kn, vn, q = chunk_inputs(w, T, lens)
    gamma = torch.from_numpy(si.gen_gamma(w)).to(dev)
    kn, vn, q = (H.to_dev(x, w, dev) for x in (kn, vn, q))
    a, b = filled(w, dev, 0, **kw), filled(w, dev, 0, **kw)
    out, sel = a.prefill(kn, vn, q, gamma)
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
    assert torch.equal(a.seq_lens, b.seq_lens)


def test_short_prefill_costs_less_than_its_steps():
    """8 positions after 126976 tokens, 4 x 8 units: 308 us against 8 steps of about
    31 when four positions always shared a wavefront, 179 now."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    T, L = 8, 126976
    cfg = spla.make_config(4, 32, 8, 128, 64, 64, 131072, n_sink=1, n_local=4)
    cache = spla.SplaCache(cfg, dev)
    g = torch.Generator(device="cuda").manual_seed(2)
    randn = lambda *s: torch.randn(s, generator=g, device=dev, dtype=torch.bfloat16)  # noqa: E731
    for _ in range(L // 15872):
        cache.append(randn(4, 8, 15872, 128), randn(4, 8, 15872, 128))
    kn, vn, q = randn(T, 4, 8, 128), randn(T, 4, 8, 128), randn(T, 4, 32, 128)
    gamma = torch.ones((32, 128), device=dev)
    n0 = cache.seq_lens.clone()

    def best(call):
        took = 1e9
        for _ in range(8):
            cache.seq_lens.copy_(n0)
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            call()
            b.record()
            torch.cuda.synchronize()
            took = min(took, a.elapsed_time(b) * 1e3)
        return took

    def step_by_step():
        for t in range(T):
            cache.step(kn[t], vn[t], q[t], gamma)

    one, many = best(lambda: cache.prefill(kn, vn, q, gamma)), best(step_by_step)
    H.log(f"{T} positions: prefill {one:.1f} us, steps {many:.1f} us")
    assert one < many, (one, many)
