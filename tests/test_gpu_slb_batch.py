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


# The kernels and the map of workgroups to tools change with the sizes of a batch: registries of one range, of
# fewer ranges than the chip has XCDs and of more, around the sizes where lists take over from tile
# maxima, ragged last tiles, blocks and query blocks.
@pytest.mark.parametrize("n_tools,n_q,k,dim", [
    (300, 1279, 2, 768), (300, 1280, 2, 768), (700, 1399, 3, 512), (700, 1400, 4, 512), (999, 3000, 8, 512),
    (1001, 3000, 8, 512), (250, 16384, 3, 512), (129, 16400, 1, 576), (128, 16400, 1, 576), (5601, 1400, 3, 576),
    (5599, 1400, 3, 576), (2049, 4100, 4, 64), (2050, 4100, 4, 64), (257, 8200, 8, 64), (5000, 600, 8, 192),
    (2000, 3000, 8, 64), (4096, 2000, 5, 128), (9000, 1100, 1, 256), (65, 16400, 4, 832), (193, 32800, 8, 832),
    (200, 32768, 3, 320),
])
def test_large_batches(n_tools, n_q, k, dim):
    import oracle as O
    from paper_2608_20397_amd import nexus as N
    rng = np.random.default_rng(n_tools + n_q)
    rtq = rng.integers(-127, 128, (n_tools, dim)).astype(np.int8)
    rtq[n_tools // 2:] = rtq[:n_tools - n_tools // 2]            # equal scores across tiles and ranges
    rts = np.full(n_tools, 0.004, np.float32)
    rqq = rng.integers(-127, 128, (n_q, dim)).astype(np.int8)
    rqs = rng.uniform(0.001, 0.01, n_q).astype(np.float32)
    d = lambda x: torch.from_numpy(x).cuda()
    idx, score, margin, route = N.slb_scan(d(rtq), d(rts), d(rqq), d(rqs), k, 1e-3)
    torch.cuda.synchronize()
    sel = np.unique(np.r_[0:20, 60:70, n_q // 2:n_q // 2 + 20, n_q - 40:n_q])
    ridx, rscore, rmargin, rroute = O.slb_scan(rtq, rts, rqq[sel], rqs[sel], k, 1e-3)
    assert np.array_equal(idx.cpu().numpy()[sel], ridx)
    assert np.array_equal(score.cpu().numpy()[sel].view(np.uint32), rscore.view(np.uint32))
    assert np.array_equal(margin.cpu().numpy()[sel].view(np.uint32), rmargin.view(np.uint32))
    assert np.array_equal(route.cpu().numpy()[sel], rroute)
