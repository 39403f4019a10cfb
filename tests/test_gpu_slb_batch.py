"""GPU parity of the batched SLB scan (tile maxima, then the best tiles scored again) against the
oracle, bit for bit, where the choice of tiles can go wrong: scores all equal, registries sorted by
score in either direction, runs of equal scores across tile and block edges, zero queries, negative scales,
registries around one range and of ragged tiles, batches around a query block, and a batch that goes in
two chunks over a million tools."""

import numpy as np
import pytest
import torch

from test_gpu_slb import _check_scan

pytestmark = pytest.mark.gpu


def _check(rtq, rts, rqq, rqs, k, tag):
    d = lambda x: torch.from_numpy(x).cuda()
    _check_scan(d(rtq), d(rts), d(rqq), d(rqs), k, 1e-3, rtq, rts, rqq, rqs, tag)


@pytest.mark.parametrize("order", ["equal", "rising", "falling", "runs", "zero", "negative"])
@pytest.mark.parametrize("n_tools,n_q,k", [(256, 17, 3), (257, 17, 8), (1000, 65, 2),
                                           (4099, 64, 8), (20000, 33, 4)])
def test_tile_choice(order, n_tools, n_q, k):
    rng = np.random.default_rng(n_tools + k)
    dim = 128
    rtq = rng.integers(-127, 128, (n_tools, dim)).astype(np.int8)
    rts = rng.uniform(0.001, 0.01, n_tools).astype(np.float32)
    rqq = rng.integers(-127, 128, (n_q, dim)).astype(np.int8)
    rqs = rng.uniform(0.001, 0.01, n_q).astype(np.float32)
    if order != "zero" and order != "negative":
        rtq[:] = rtq[0]
        rqq[: n_q // 2] = rtq[0]                          # positive scores, negative ones below
        rqq[n_q // 2:] = -rtq[0]
        i = np.arange(n_tools, dtype=np.float32)
        rts = {"equal": np.full(n_tools, 0.004, np.float32), "rising": (1 + i) * np.float32(1e-4),
               "falling": (n_tools - i) * np.float32(1e-4),
               "runs": (1 + (i // 5) % 7).astype(np.float32)}[order]
    elif order == "zero":
        rqq[::4] = 0                                      # every score +0
    else:
        rts[::2] *= -1
        rqs[::3] *= -1
    _check(rtq, rts, rqq, rqs, k, f"{order} {n_tools}x{n_q} k{k}")


def test_chunks_of_queries():
    """2^20 tools take 256 queries a pass: 300 queries go in two."""
    rng = np.random.default_rng(5)
    n_tools, n_q, dim, k = 1 << 20, 300, 64, 5
    rtq = rng.integers(-127, 128, (n_tools, dim)).astype(np.int8)
    rts = rng.uniform(0.001, 0.01, n_tools).astype(np.float32)
    rqq = rng.integers(-127, 128, (n_q, dim)).astype(np.int8)
    rqs = rng.uniform(0.001, 0.01, n_q).astype(np.float32)
    import oracle as O
    from paper_2608_20397_amd import nexus as N
    d = lambda x: torch.from_numpy(x).cuda()
    idx, score, margin, route = N.slb_scan(d(rtq), d(rts), d(rqq), d(rqs), k, 1e-3)
    torch.cuda.synchronize()
    sel = np.array([0, 64, 255, 256, 299])
    ridx, rscore, rmargin, rroute = O.slb_scan(rtq, rts, rqq[sel], rqs[sel], k, 1e-3)
    assert np.array_equal(idx.cpu().numpy()[sel], ridx)
    assert np.array_equal(score.cpu().numpy()[sel].view(np.uint32), rscore.view(np.uint32))
    assert np.array_equal(margin.cpu().numpy()[sel].view(np.uint32), rmargin.view(np.uint32))
    assert np.array_equal(route.cpu().numpy()[sel], rroute)
