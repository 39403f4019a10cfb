"""GPU parity of the head_dim-64 row-major attention against the fp64 oracle at the edges of its tiles
(64 keys, 32 queries, 16-token pages): every row and head, one to 32 query heads per KV head, with and
without the soft cap, shuffled pages, NaN in every slot past the sequence."""

import numpy as np
import pytest
import torch

import oracle as O
from paper_2608_20397_amd import nexus as N
from synth import PAGE
from synth import gen as G

from _pipeline import BF16_MAX_ABS, BF16_REL_RMS, compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_kv,g,cap", [(3, 1, 0.0), (2, 3, 50.0), (1, 32, 0.0)])
@pytest.mark.parametrize("n_s,n_past", [(1, 0), (1, 63), (31, 1), (33, 30), (64, 64), (65, 127),
                                        (5, 1018), (300, 0), (130, 2111)])
def test_d64_edges(n_kv, g, cap, n_s, n_past):
    d, n_tok = 64, n_s + n_past
    n_log = (n_tok + PAGE - 1) // PAGE
    npp = n_log + 3
    std = d ** -0.5
    k = G.device_normal(2, n_s, 1, (1, npp, n_kv, PAGE, d), 1.0, "bf16", "cuda")
    v = G.device_normal(2, n_s, 2, (1, npp, n_kv, PAGE, d), std, "bf16", "cuda")
    pm = np.random.default_rng([n_s, n_past]).permutation(npp)[:n_log].astype(np.int32)
    spare = np.setdiff1d(np.arange(npp), pm)
    for x in (k, v):
        x[:, torch.from_numpy(spare).cuda()] = float("nan")
        x[:, int(pm[-1]), :, (n_tok - 1) % PAGE + 1:] = float("nan")
    cache = N.PagedKVCache(k, v, torch.from_numpy(pm).cuda(), 1e4)
    q = G.device_normal(2, n_past, 0, (n_s, n_kv * g, d), std, "bf16", "cuda")
    out = N.suffix_attn(q, cache, 0, n_past, softcap=cap)
    torch.cuda.synchronize()
    lk, lv = O.gather_logical(G.torch_to_bits(k), G.torch_to_bits(v), pm, n_tok, PAGE, O.ROWMAJOR)
    ref = O.suffix_attention(O.storage_to_f64(G.torch_to_bits(q), "bf16"),
                             O.storage_to_f64(lk[0], "bf16"), O.storage_to_f64(lv[0], "bf16"),
                             n_past, softcap=cap)
    got = O.bf16_bits_to_f64(G.torch_to_bits(out))
    assert np.isfinite(got).all()
    ma, rr = compare(got, ref)
    print(f"max-abs {ma:.3e} rel-RMS {rr:.3e}", flush=True)
    assert ma <= BF16_MAX_ABS and rr <= BF16_REL_RMS, (ma, rr)
