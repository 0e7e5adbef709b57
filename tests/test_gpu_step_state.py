"""The state that a step leaves does not depend on who applies the token's update: the
sparse pass (8 workgroups per head, in one launch or apart) or the single-token
append (groups of more than 8 heads), over the same keys and values."""

import numpy as np
import pytest
import torch

import gpu_harness as H
import spla_inputs as si
from paper_2601_22379_amd import spla

pytestmark = pytest.mark.gpu


def test_same_bits_as_the_append():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    states = []
    for group, flags in ((4, 0), (4, spla.FLAG_SEPARATE_KERNELS), (12, 0)):
        w = si.custom("stepstate", 2, 4 * group, 4, 128, 64, 16, [1500, 777], kind="iid", code=350,
                      capacity=2048)
        cache = spla.SplaCache(H.config_of(w, flags=flags), dev)
        H.fill_cache(w, cache, device=dev)
        rng = np.random.default_rng(8)
        gamma = torch.from_numpy(si.gen_gamma(w)).to(dev)
        for t in range(5):
            kn, vn = (H.to_dev(3 * rng.standard_normal((w.batch, 4, 128)), w, dev)
                      for _ in range(2))
            cache.step(kn, vn, H.to_dev(si.gen_q_batch(w, t), w, dev), gamma)
        torch.cuda.synchronize()
        states.append((cache.state, cache.norm, cache.stats, cache.seq_lens))
    for other in states[1:]:
        for x, y in zip(states[0], other):
            assert torch.equal(x, y), (x - y).abs().max()
