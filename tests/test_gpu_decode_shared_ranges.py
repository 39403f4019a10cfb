"""GPU parity of the decode step over physical pages that sequences share, at lengths for which the launch
takes them together (512 MB of keys and values or more), against the fp64 oracle on sampled sequences;
tolerances as the other decode tests.  The shared pages span many ranges.

A value that is not finite belongs to the sequences that map its page: every other sequence of the
batch must come out as if it were not there."""

import numpy as np
import pytest
import torch

import oracle as O
from paper_2608_20397_amd import nexus as N
from synth import PAGE

from test_gpu_decode import _check

pytestmark = pytest.mark.gpu


class Batch:
    """Sequences of lens[b] tokens over one pool; those listed in share = [(sequences, pages)] map the first
    pages of the first of them, except the (sequence, page) pairs of `moved`."""

    def __init__(self, d, kv, g, lens, share, layout="rowmajor", cap=0.0, moved=(), seed=1):
        self.layout, self.cap, self.lens = layout, cap, list(lens)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        pages = [-(-n // PAGE) for n in lens]
        first = np.cumsum([0] + pages)
        maps = np.zeros((len(lens), max(pages)), dtype=np.int64)
        for b, n in enumerate(pages):
            maps[b, :n] = first[b] + np.arange(n)
        for seqs, n in share:
            for b in seqs[1:]:
                keep = [p for p in range(min(n, lens[b] // PAGE)) if (b, p) not in moved]
                maps[b, keep] = maps[seqs[0], keep]
        used = np.unique(np.concatenate([maps[b, :n] for b, n in enumerate(pages)]))
        place = np.random.default_rng(seed).permutation(len(used))
        self.maps = place[np.searchsorted(used, maps).clip(max=len(used) - 1)].astype(np.int32)
        npp = len(used)
        normal = lambda shape, std: (torch.randn(shape, generator=gen, device="cuda") * std).bfloat16()
        self.k = normal((1, npp, kv, PAGE, d), 2 * d ** -0.5)
        self.v = normal((1, kv, d, npp * PAGE) if layout == "transposed" else self.k.shape, 1.0)
        self.q = normal((len(lens), kv * g, d), 1.0)
        self.bytes = len(lens) * max(lens) * kv * d * 4   # the launch's bound

    def values(self, b, p):
        """V of sequence b's page p, every head."""
        phys = int(self.maps[b, p])
        if self.layout == "transposed":
            return self.v[0, :, :, phys * PAGE:(phys + 1) * PAGE]
        return self.v[0, phys]

    def run(self, **kw):
        cache = N.PagedKVCache(self.k, self.v, torch.zeros(1, dtype=torch.int32, device="cuda"), 1e4,
                               N.V_TRANSPOSED if self.layout == "transposed" else N.V_ROWMAJOR)
        out = N.decode_attn(self.q, cache, torch.from_numpy(self.maps).cuda(),
                            torch.tensor(self.lens, dtype=torch.int32, device="cuda"), max(self.lens),
                            0, softcap=self.cap, **kw)
        torch.cuda.synchronize()
        return out.float().cpu().double().numpy()

    def oracle(self, seqs):
        f64 = lambda x: x.float().cpu().double().numpy()
        return O.decode_attention(f64(self.q)[seqs], f64(self.k[0]), f64(self.v[0]), self.maps[seqs],
                                  [self.lens[b] for b in seqs], PAGE, self.layout, softcap=self.cap)


SHAPES = [
    # head_dim, KV heads, query heads per KV head, V layout, cap, sequences, tokens, shared pages
    (128, 8, 5, "rowmajor", 0.0, 9, 15000, 800),
    (256, 8, 2, "transposed", 50.0, 6, 11200, 650),
    (64, 2, 32, "rowmajor", 0.0, 16, 66200, 4096),
    (128, 8, 3, "transposed", 0.0, 17, 8200, 333),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"d{s[0]}-{s[3]}")
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_nonfinite_values_stay_with_their_sequences(shape, bad):
    d, kv, g, layout, cap, n, tokens, shared = shape
    lens = [tokens - 37 * b for b in range(n)]
    # page 40 is shared by the first two sequences alone, page 41 by the last two
    moved = [(b, 40) for b in range(2, n)] + [(b, 41) for b in range(1, n)]
    t = Batch(d, kv, g, lens, [(range(n), shared)], layout, cap, moved)
    t.maps[n - 2, 41] = t.maps[n - 1, 41]
    assert t.bytes >= 512 << 20
    print(f"decode {shape}: values {bad}", flush=True)
    hit = [0, 1, 3]
    t.values(0, shared + 3)[:] = bad           # private to the first sequence, behind the prefix
    t.values(3, shared + 1)[:] = bad           # to a later one
    t.values(0, 40)[:] = bad                   # of the first two
    got = t.run()
    assert not np.isfinite(got[hit]).any()
    others = [b for b in range(n) if b not in hit]
    assert np.isfinite(got[others]).all()
    sel = [2, others[len(others) // 2], n - 1]
    _check(got[sel], t.oracle(sel), "bf16", f"{shape}")



A, E, O_ = range(9), range(0, 32, 2), range(1, 32, 2)
CASES = {
    # head_dim, KV heads, query heads per KV head, V layout, cap, tokens, shares, moved, sequences that share
    "range edges, middle pages elsewhere": (
        128, 8, 5, "rowmajor", 0.0, [15000 - 300 * b for b in A], [(A, 640)],
        [(2, p) for p in range(100, 140)] + [(5, 31), (5, 32), (8, 639)], A),
    "prefix inside a range, cap": (
        128, 8, 5, "rowmajor", 30.0, [15000 - 300 * b for b in A], [(A, 777)], [(0, 300)], A),
    "short ones beside, a short representative": (
        64, 8, 4, "transposed", 0.0,
        [0, 7000, 15, 16, 9000, 2000, 3400] + [12000 - 100 * i for i in range(20)],
        [([1, 4] + list(range(7, 27)), 437)], [(1, 9)], [1, 4] + list(range(7, 27))),
    "two groups of 12, one head a column block": (
        128, 2, 16, "transposed", 0.0, [24000 + b for b in range(24)], [(range(12), 1000), (range(12, 24), 900)],
        [], range(24)),
    "one group shares, one has a private sequence": (
        128, 2, 20, "rowmajor", 0.0, [24000 + b for b in range(24)], [(range(23), 1400)], [], range(12)),
    "interleaved prefixes share nothing": (
        128, 8, 2, "rowmajor", 0.0, [4500] * 32, [(E, 270), (O_, 270)], [], []),
    "one page shares nothing": (256, 8, 2, "rowmajor", 50.0, [9000] * 8, [(range(8), 1)], [], []),
    "a page more than half": (256, 8, 1, "rowmajor", 0.0, [9000] * 8, [(range(8), 282)], [], range(8)),
    "half": (256, 8, 1, "transposed", 0.0, [9000] * 8, [(range(8), 281)], [], []),
    "everything": (128, 8, 1, "rowmajor", 0.0, [16 * 280] * 33, [(range(33), 280)], [], range(33)),
}


@pytest.mark.parametrize("name", CASES)
def test_ranges(name):
    d, kv, g, layout, cap, lens, share, moved, sharers = CASES[name]
    t = Batch(d, kv, g, lens, share, layout, cap, moved)
    assert t.bytes >= 512 << 20
    print(name, flush=True)
    ranges, got = _run_in(t, _bytes(t))
    print("ranges", ranges, flush=True)
    assert [b for b, r in enumerate(ranges) if r > 0] == list(sharers)
    sel = sorted({0, 1, 2, len(lens) // 2, len(lens) - 1} | {b for b, _ in moved})
    _check(got[sel], t.oracle(sel), "bf16", name)


def _bytes(t):
    cache = N.PagedKVCache(t.k, t.v, torch.zeros(1, dtype=torch.int32, device="cuda"), 1e4,
                           N.V_TRANSPOSED if t.layout == "transposed" else N.V_ROWMAJOR)
    return N.decode_attn_workspace_bytes(cache, len(t.lens), t.q.shape[1], max(t.lens))


def _run_in(t, nbytes):
    """(ranges of shared pages that each sequence has partials of, output): the former are the last
    entries of a workspace that the call fills."""
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
    got = t.run(workspace=ws)
    n = len(t.lens)
    return ws[nbytes - 4 * n:].view(torch.int32).tolist(), got


@pytest.mark.parametrize("ranges", [4, 5, 6])
def test_ranges_of_a_small_workspace(ranges):
    """Ranges as long as a workgroup's lists hold (1024 pages) where the workspace has few partials; with
    too few even for those nothing is shared."""
    d, kv, g, n, tokens = 64, 2, 3, 16, 66200
    t = Batch(d, kv, g, [tokens - 50 * b for b in range(n)], [(range(n), 4000)],
              moved=[(3, 827), (3, 828), (4, 3500)])
    rows = n * kv * g * (d + 2) * 4
    pages = -(-tokens // PAGE)
    sp = -(-pages // 16)
    splits = -(-pages // sp)
    nbytes = rows * (splits + ranges) + 4 * n
    got_ranges, got = _run_in(t, nbytes)
    print(got_ranges, flush=True)
    if ranges >= 5:
        assert got_ranges == [ranges] * n
    sel = [0, 3, 4, n - 1]
    _check(got[sel], t.oracle(sel), "bf16", f"{ranges} ranges")


@pytest.mark.parametrize("d,layout", [(64, "rowmajor"), (128, "rowmajor"), (128, "transposed"),
                                      (256, "rowmajor")])
@pytest.mark.parametrize("pages", [1, 4, 5, 33])
def test_infinite_value_in_a_page_without_a_pair(d, layout, pages):
    """Pages are taken two at a time: an odd one's infinity comes out as the infinity it is."""
    t = Batch(d, 2, 3, [PAGE * pages], [], layout)
    for p in range(pages):
        v = t.values(0, p).clone()
        if layout == "transposed":
            t.values(0, p)[:, 5, 3] = float("inf")
        else:
            t.values(0, p)[:, 3, 5] = float("inf")
        got = t.run()
        assert np.isposinf(got[..., 5]).all(), p
        t.values(0, p)[:] = v


def test_one_workspace_for_all_smaller_batches():
    """A buffer sized for the largest batch serves every smaller one, across the edge of a group (32
    sequences) on both sides of which the shared pages' partials differ, and so does one that holds
    nothing beside the partials of the sequences' own pages; one byte less than those is refused."""
    d, kv, g, tokens = 128, 8, 5, 4400
    for largest in (33, 48):
        t = Batch(d, kv, g, [tokens] * largest, [(range(largest), 260)])
        cache = N.PagedKVCache(t.k, t.v, torch.zeros(1, dtype=torch.int32, device="cuda"), 1e4)
        size = lambda n: N.decode_attn_workspace_bytes(cache, n, kv * g, tokens)
        buf = torch.empty(size(largest), dtype=torch.uint8, device="cuda")
        if largest == 33:
            assert size(32) > buf.numel()
        full, maps, q = t.oracle(range(largest)), t.maps, t.q
        for n in (2, 31, 32, 33, 48):
            if n > largest:
                continue
            t.lens, t.maps, t.q = [tokens] * n, np.ascontiguousarray(maps[:n]), q[:n].contiguous()
            for ws in (buf, buf[:_own_bytes(n, kv, g, d, tokens)]):
                buf.fill_(0xFF)
                _check(t.run(workspace=ws), full[:n], "bf16", f"{n} sequences, {ws.numel()} bytes")
            with pytest.raises(N.NexusError) as e:
                t.run(workspace=buf[:_own_bytes(n, kv, g, d, tokens) - 1])
            assert e.value.status == N.EWORKSPACE


def _own_bytes(n, kv, g, d, tokens):
    """Partials of the sequences' own splits (tests of up to 256 workgroup pairs)."""
    pages, pairs = -(-tokens // PAGE), n * kv
    sp = max(-(-pages // -(-512 // pairs)), 32)
    splits = -(-pages // sp)
    if 256 < pairs * splits < 512 and pairs <= 256:
        splits = 256 // pairs
        splits = -(-pages // -(-pages // splits))
    return n * kv * g * splits * (d + 2) * 4 if splits > 1 else 1


@pytest.mark.parametrize("d,kv,layout,n,tokens", [(128, 8, "rowmajor", 9, 15000), (64, 2, "transposed", 3, 900),
                                                  (256, 8, "transposed", 1, 2000)])
def test_cache_base_not_16_byte_aligned(d, kv, layout, n, tokens):
    """A cache that starts 2 bytes past a 16-byte boundary, with and without shared pages to look for."""
    t = Batch(d, kv, 3, [tokens - 20 * b for b in range(n)], [(range(n), tokens // 20)], layout)
    for name in ("k", "v"):
        x = getattr(t, name)
        pool = torch.zeros(x.numel() + 8, dtype=x.dtype, device="cuda")
        y = pool[1:1 + x.numel()].view(x.shape)
        y.copy_(x)
        assert y.data_ptr() % 16 == 2
        setattr(t, name, y)
    sel = sorted({0, n // 2, n - 1})
    _check(t.run()[sel], t.oracle(sel), "bf16", f"head_dim {d} {layout}, base at 2 bytes")
