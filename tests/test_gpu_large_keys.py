"""Keys whose exponentials overflow, or vanish, unless phi(k) is taken relative
to the row's maximum: the fused pass against the oracle, one launch and
separate launches. Steps with ordinary keys lie between the others."""

import pytest
import torch

import gpu_harness as H
import spla_inputs as si
from paper_2601_22379_amd import spla

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [120.0, -120.0])
@pytest.mark.parametrize("flags,n_q", [(0, 4), (spla.FLAG_SEPARATE_KERNELS, 4), (0, 8)])
def test_decode_with_large_keys(flags, n_q, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    w = si.custom("large", 1, n_q, 1, 128, 64, 6, [1205], kind="block_offsets", code=280,
                  offset_std=0.5)
    cache = spla.SplaCache(H.config_of(w, flags=flags), dev)
    K, V, n = si.gen_kv_slab(w, 0, 1205)
    K[:, :, 300:] = si.round_bf16(K[:, :, 300:] + shift)  # blocks before and after the change
    cache.append(H.to_dev(K, w, dev), H.to_dev(V, w, dev), torch.from_numpy(n).to(dev))
    q, gamma = si.gen_q_batch(w), si.gen_gamma(w)
    out, sel = cache.decode(H.to_dev(q, w, dev), torch.from_numpy(gamma).to(dev))
    torch.cuda.synchronize()
    import oracle as O
    r = O.decode_sequence(q[0], K[0], V[0], 1205, gamma, H.params_of(w))[0]
    assert sel[0, 0].tolist()[:len(r.sel)] == list(r.sel)
    got = out[0].float().cpu().numpy()
    err = (abs(got - r.out).max(axis=1) / abs(r.out).max(axis=1)).max()
    assert err < H.TOL["bf16"], err
