"""GPU parity of the fp32 suffix attention against the fp64 oracle where its kernel can go wrong:
every head_dim it is built for, both V layouts, the cap on and off, rows (query, head of the
group) that fill, straddle and leave part of a 16-row tile, contexts of less than one page, of a
page per wave and one more, and many.  Tolerance as the other fp32 attention tests."""

import numpy as np
import pytest
import torch

from paper_2608_20397_amd import nexus as N
from synth import gen as G

from _pipeline import VL, custom_workload, oracle_attention, oracle_cache, to_f64
from test_gpu_attention import _check

pytestmark = pytest.mark.gpu

# head_dim, KV heads, group, context, block, user tokens, suffix, V layout, cap, shuffled
CASES = [
    (8, 1, 1, 0, 1, 0, 1, "rowmajor", 0.0, False),
    (8, 2, 3, 100, 30, 7, 33, "transposed", 20.0, True),
    (16, 1, 5, 15, 2, 0, 2, "rowmajor", 30.0, False),
    (16, 2, 1, 200, 17, 0, 17, "transposed", 0.0, True),
    (32, 3, 2, 63, 40, 1, 41, "rowmajor", 0.0, True),
    (64, 1, 16, 126, 2, 0, 1, "transposed", 0.0, False),
    (64, 2, 17, 129, 16, 0, 3, "rowmajor", 5.0, True),
    (128, 2, 5, 127, 20, 0, 16, "rowmajor", 0.0, True),
    (128, 1, 5, 1000, 33, 8, 40, "transposed", 50.0, True),
    (256, 2, 2, 64, 9, 0, 9, "rowmajor", 50.0, False),
    (256, 1, 3, 65, 21, 0, 21, "transposed", 0.0, True),
]


def _run(i, change=None):
    """(got, ref) of case i over the oracle's cache; ``change`` edits the device cache first."""
    d, kv, g, n_ctx, block, user, suffix, layout, cap, shuffled = CASES[i]
    wl = custom_workload(1, n_ctx, block, user, suffix, head_dim=d, n_kv_heads=kv,
                         n_q_heads=kv * g, v_layout=layout, softcap=cap, shuffled_pages=shuffled)
    hc = G.host_case_wl(wl, 700 + i)
    ck, cv = oracle_cache(hc)
    cache = N.PagedKVCache(G.bits_to_torch(ck, "f32", "cuda"), G.bits_to_torch(cv, "f32", "cuda"),
                           torch.from_numpy(hc.page_map).cuda(), wl.rope_base, VL[layout])
    if change is not None:
        change(wl, hc.page_map, cache)
    q = G.bits_to_torch(hc.q[0], "f32", "cuda")
    out = N.suffix_attn(q, cache, 0, wl.attn_n_past[0], wl.softcap)
    torch.cuda.synchronize()
    return to_f64(out), oracle_attention(hc, ck, cv, 0)


@pytest.mark.parametrize("i", range(len(CASES)))
def test_f32_shapes(i):
    print(f"f32 {CASES[i]}", flush=True)
    got, ref = _run(i)
    _check(got, ref, "f32", f"f32 {CASES[i]}")


# A value row with an infinity or a NaN reaches the queries that see its token and no others.
@pytest.mark.parametrize("i", [4, 7, 8, 10])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_f32_nonfinite_value_stays_causal(i, bad):
    print(f"f32 {CASES[i]}: value {bad} three tokens from the end", flush=True)

    def change(wl, page_map, cache):
        t = wl.n_tokens - 3
        page, slot = int(page_map[t // 16]), t % 16
        if wl.v_layout == "transposed":
            cache.v[0, :, :, page * 16 + slot] = bad
        else:
            cache.v[0, page, :, slot] = bad

    got, ref = _run(i, change)
    _check(got[:-3], ref[:-3], "f32", f"f32 {CASES[i]} rows before the token")
    assert not np.isfinite(got[-3:]).any()
