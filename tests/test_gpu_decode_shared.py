"""GPU parity of the decode step where sequences share physical pages in a launch whose bound on the
sequences' keys and values is 512 MB or more, so that it looks for such pages, while the lengths are far
below it, so that it reads them sequence by sequence all the same: lengths 0 and below one page, sequences
that leave a shared prefix for a page and come back, 1 to 32 query heads per KV head, groups of every
fill, a group more than one, both V layouts, the cap.  (Lengths at which the pages are taken together:
test_gpu_decode_shared_ranges.)  Against the fp64 oracle, tolerances as the other decode tests."""

import dataclasses

import pytest
import torch

from paper_2608_20397_amd import nexus as N
from synth import PAGE
from synth import decode as SD

from test_gpu_decode import _check, _oracle, _upload

pytestmark = pytest.mark.gpu

# head_dim, KV heads, group, lengths, shared prefix, V layout, cap, pages (sequence, page) that a
# sequence maps elsewhere
CASES = [
    (128, 8, 5, [300, 289, 272, 500, 257, 256, 600], 256, "rowmajor", 0.0, []),
    (128, 2, 5, [40 + 9 * i for i in range(40)], 32, "rowmajor", 30.0, [(3, 1), (11, 0), (39, 0)]),
    (128, 2, 16, [900, 700, 650, 641], 640, "transposed", 0.0, [(1, 5), (1, 6), (3, 39)]),
    (64, 2, 1, [0, 15, 530, 700, 560, 16, 0, 531], 512, "rowmajor", 0.0, [(3, 0), (4, 31)]),
    (64, 2, 32, [1200, 1100, 1033], 1024, "rowmajor", 20.0, [(2, 17)]),
    (256, 2, 2, [200, 333, 180, 161, 170], 160, "transposed", 50.0, [(0, 3), (4, 9)]),
    (256, 1, 8, [97, 1500, 700], 96, "rowmajor", 0.0, []),
    (64, 4, 4, [100, 200, 300, 400], 0, "transposed", 0.0, []),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_shared_pages(i):
    d, kv, g, lens, prefix, layout, cap, moved = CASES[i]
    print(f"shared decode {CASES[i]}", flush=True)
    wl = dataclasses.replace(
        SD.decode_workload(2), case=1200 + i, name=f"shared {i}", n_q_heads=g * kv, n_kv_heads=kv,
        head_dim=d, lens=tuple(lens), shared_prefix=0, v_layout=layout, softcap=cap,
        shuffled=True, q_scale=1.0, k_scale=d ** -0.5 * 2, v_scale=1.0)
    hc = SD.decode_host_case_wl(wl)
    # share: the first pages of every sequence become those of the longest one
    src = max(range(len(lens)), key=lambda b: lens[b])
    for b, n in enumerate(lens):
        for p in range(min(prefix, n) // PAGE):
            if (b, p) not in moved:
                hc.maps[b, p] = hc.maps[src, p]
    cache, _, dlens, q = _upload(hc)
    # the bound that makes the launch look for shared pages, and map rows that long
    bound = -(-(512 << 20) // (len(lens) * kv * d * 4))
    stride = -(-bound // PAGE)
    maps = torch.zeros((len(lens), stride), dtype=torch.int32)
    maps[:, :hc.maps.shape[1]] = torch.from_numpy(hc.maps).clamp(min=0)
    out = N.decode_attn(q[0], cache, maps.cuda(), dlens, bound, 0, softcap=cap)
    torch.cuda.synchronize()
    got = out.float().cpu().double().numpy()
    _check(got, _oracle(hc, 0), "bf16", f"shared decode {CASES[i]}")
    for b, n in enumerate(lens):
        if n == 0:
            assert not got[b].any(), b
