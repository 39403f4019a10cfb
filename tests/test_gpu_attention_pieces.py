"""GPU parity of one-suffix attention against the fp64 oracle, every row and head, where its key axis is
cut finest and its tails are shortest: few queries in up to 17 pieces of 256 keys (more than the
combine reads at once), and last tiles of one to 63 keys.  head_dim 64, 128 and 256, row-major and
transposed V with NaN in every slot past the sequence and in every page it does not map."""

import numpy as np
import pytest
import torch

import oracle as O
from paper_2608_20397_amd import nexus as N
from synth import PAGE
from synth import gen as G

from _pipeline import BF16_MAX_ABS, BF16_REL_RMS, compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,vt,cap", [(64, False, 0.0), (64, True, 50.0), (128, False, 0.0),
                                      (128, True, 0.0), (128, True, 50.0), (256, False, 50.0),
                                      (256, True, 50.0)])
@pytest.mark.parametrize("n_s,n_past", [(1, 0), (7, 2), (1, 4098), (16, 2025), (33, 1103), (70, 1000),
                                        (200, 2488), (127, 64), (300, 20)])
def test_pieces(d, vt, cap, n_s, n_past):
    n_kv, g, n_tok = 2, 3, n_s + n_past
    n_log = (n_tok + PAGE - 1) // PAGE
    npp = n_log + 3
    std = d ** -0.5
    k = G.device_normal(2, n_s, 1, (1, npp, n_kv, PAGE, d), 1.0, "bf16", "cuda")
    vshape = (1, n_kv, d, npp * PAGE) if vt else (1, npp, n_kv, PAGE, d)
    v = G.device_normal(2, n_s, 2, vshape, std, "bf16", "cuda")
    pm = np.random.default_rng([n_s, n_past, d]).permutation(npp)[:n_log].astype(np.int32)
    spare = torch.from_numpy(np.setdiff1d(np.arange(npp), pm)).cuda()
    last, used = int(pm[-1]), (n_tok - 1) % PAGE + 1
    vp = v.view(1, n_kv, d, npp, PAGE) if vt else v
    k[:, spare] = float("nan")
    k[:, last, :, used:] = float("nan")
    if vt:
        vp[:, :, :, spare] = float("nan")
        vp[:, :, :, last, used:] = float("nan")
    else:
        vp[:, spare] = float("nan")
        vp[:, last, :, used:] = float("nan")
    cache = N.PagedKVCache(k, v, torch.from_numpy(pm).cuda(), 1e4,
                           N.V_TRANSPOSED if vt else N.V_ROWMAJOR)
    q = G.device_normal(2, n_past, 0, (n_s, n_kv * g, d), std, "bf16", "cuda")
    out = N.suffix_attn(q, cache, 0, n_past, softcap=cap)
    torch.cuda.synchronize()
    lk, lv = O.gather_logical(G.torch_to_bits(k), G.torch_to_bits(v), pm, n_tok, PAGE,
                              O.TRANSPOSED if vt else O.ROWMAJOR)
    ref = O.suffix_attention(O.storage_to_f64(G.torch_to_bits(q), "bf16"),
                             O.storage_to_f64(lk[0], "bf16"), O.storage_to_f64(lv[0], "bf16"),
                             n_past, softcap=cap)
    got = O.bf16_bits_to_f64(G.torch_to_bits(out))
    assert np.isfinite(got).all()
    ma, rr = compare(got, ref)
    print(f"max-abs {ma:.3e} rel-RMS {rr:.3e}", flush=True)
    assert ma <= BF16_MAX_ABS and rr <= BF16_REL_RMS, (ma, rr)


@pytest.mark.parametrize("d,vt", [(64, False), (64, True), (128, False), (128, True), (256, False), (256, True)])
def test_cache_base_not_16_byte_aligned(d, vt):
    """The same bits from a cache that starts 2 bytes past a 16-byte boundary."""
    n_kv, g, n_s, n_past = 2, 2, 75, 700
    npp = (n_s + n_past + PAGE - 1) // PAGE
    shape = (1, npp, n_kv, PAGE, d)
    k = G.device_normal(2, 1, 1, shape, 1.0, "bf16", "cuda")
    v = G.device_normal(2, 1, 2, (1, n_kv, d, npp * PAGE) if vt else shape, 0.1, "bf16", "cuda")
    q = G.device_normal(2, 1, 0, (n_s, n_kv * g, d), 0.1, "bf16", "cuda")
    pm = torch.from_numpy(np.random.default_rng(3).permutation(npp).astype(np.int32)).cuda()
    outs = []
    for shift in (0, 1):
        moved = []
        for x in (k, v):
            pool = torch.zeros(x.numel() + 8, dtype=x.dtype, device="cuda")
            y = pool[shift:shift + x.numel()].view(x.shape)
            y.copy_(x)
            moved.append(y)
        cache = N.PagedKVCache(*moved, pm, 1e4, N.V_TRANSPOSED if vt else N.V_ROWMAJOR)
        outs.append(N.suffix_attn(q, cache, 0, n_past))
        torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
