"""GPU parity of the splice into a transposed V cache against the oracle, bit for bit over the whole
cache, at the edges of the thread blocks (8 tokens in bf16, 4 in f32), pages and workgroups: offsets and
lengths that cut a block at either end or lie inside one, head counts that fill no round of 8 groups,
the smallest and largest rows."""

import numpy as np
import pytest
import torch

import oracle as O
from paper_2608_20397_amd import nexus as N
from synth import PAGE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 16), ("bf16", 64), ("bf16", 256), ("f32", 8),
                                     ("f32", 128)])
@pytest.mark.parametrize("layers,heads", [(1, 1), (3, 3), (2, 8)])
@pytest.mark.parametrize("offset,n", [(0, 1), (7, 1), (3, 2), (5, 11), (8, 8), (15, 2), (12, 100),
                                      (16, 256), (1, 143)])
def test_transposed_splice(dtype, d, layers, heads, offset, n):
    rng = np.random.default_rng([d, layers, offset, n])
    bits = np.uint16 if dtype == "bf16" else np.uint32
    tdt, ibits = (torch.bfloat16, torch.int16) if dtype == "bf16" else (torch.float32, torch.int32)
    n_log = (offset + n + PAGE - 1) // PAGE
    npp = n_log + 2
    pm = rng.permutation(npp)[:n_log].astype(np.int32)

    # finite values only: the bits then survive a view as floats
    top = 0x7F00 if dtype == "bf16" else 0x7F000000
    draw = lambda shape: rng.integers(0, top, shape).astype(bits)
    bk, bv = draw((layers, n, heads, d)), draw((layers, n, heads, d))
    ck, cv = draw((layers, npp, heads, PAGE, d)), draw((layers, heads, d, npp * PAGE))
    dev = lambda x: torch.from_numpy(x.view(np.int16 if dtype == "bf16" else np.int32).copy()) \
        .cuda().view(tdt)
    cache = N.PagedKVCache(dev(ck), dev(cv), torch.from_numpy(pm).cuda(), 1e4, N.V_TRANSPOSED)
    N.splice_pages(cache, N.Block(dev(bk), dev(bv), 0, 1e4), offset)
    torch.cuda.synchronize()
    rk, rv = O.splice_paged(ck, cv, pm, bk, bv, offset, PAGE, v_layout=O.TRANSPOSED)
    host = lambda x: x.view(ibits).cpu().numpy().view(bits)
    assert np.array_equal(host(cache.v), rv)
    assert np.array_equal(host(cache.k), rk)
