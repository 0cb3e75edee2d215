"""Gather with several environments of one capsule: how many a block serves
follows from the sizes (up to 4, 2 or 1 in launches that store more than
128 MB, 1 otherwise); every environment holds its capsule's bytes and nothing
past the boundary changes."""
import pytest
import torch

import paper_2606_20537_amd as cap

pytestmark = pytest.mark.gpu

P = 128
CASES = [
    # (row bytes, environments' ids, gallery): a capsule is 2 P rows and a small state
    (16, [0, 0, 0, 1, 1, 0], 2),                # a few tiles: a rep to each environment
    (65552, [0] * 17, 1),                       # one capsule: the same
    (8208, [1, 1, 0, 0, 0], 2),                 # 10.5 MB in all: the same
    (8160, [1, 1, 0, 0, 0], 2),
    (65552, [3, 0, 3, 1, 1, 3, 0, 3, 3], 4),    # 16.8 MB each, 151 MB in all, uneven, one capsule unused: 2, 2, 4 and 1
    (131088, [0] * 17 + [1] * 18 + [0], 2),     # 33.6 MB each: fours and rests of 2
    (24592, [i % 2 for i in range(63)] + [0, 1, 1], 2),  # 66: fours, then a second launch, of one capsule
    (24592, [i % 3 for i in range(65)], 3),     # a second launch of one
    (24592, [i % 2 for i in range(32)], 2),     # 201 MB: pairs (3096 blocks at four each)
    (8208, [i % 3 for i in range(63)], 3),      # 132.7 MB, just below 128 MiB: one each, in the caller's order
    (8208, [i % 3 for i in range(64)], 3),      # 134.8 MB, just above: pairs
    (8208, [i % 3 for i in range(70)], 3),      # and a second launch that stores little
]


@pytest.mark.parametrize("row,ids,n_gallery", CASES, ids=["%d_%d_%d" % (c[0], len(c[1]), c[2]) for c in CASES])
def test_gather_groups(row, ids, n_gallery):
    print("case", row, len(ids), n_gallery, flush=True)
    rows, state = P + 3, 4112
    gen = torch.Generator(device="cuda").manual_seed(row)

    def make():
        bufs = [torch.randint(0, 256, (rows, row), generator=gen, device="cuda", dtype=torch.uint8) for _ in range(2)]
        bufs.insert(1, torch.randint(0, 256, (1, state), generator=gen, device="cuda", dtype=torch.uint8))
        kinds = (cap.CAP_KIND_POSITIONAL, cap.CAP_KIND_FIXED, cap.CAP_KIND_POSITIONAL)
        return cap.cap_set_create([("b%d" % i, b, b.shape[1], b.shape[0], k)
                                   for i, (b, k) in enumerate(zip(bufs, kinds))], 64, 7), bufs

    gallery = []
    for _ in range(n_gallery):
        s, bufs = make()
        cap.cap_set_set_position(s, P)
        arena = torch.empty(cap.capsule_bytes(s, P), dtype=torch.uint8, device="cuda")
        gallery.append((cap.capsule_snapshot(s, P, 0, arena), bufs))
    envs = [make() for _ in ids]
    tails = [[b[P:].clone() for b in bufs] for _, bufs in envs]
    cap.capsule_gather_restore([g for g, _ in gallery], ids, [s for s, _ in envs])
    torch.cuda.synchronize()
    for (s, bufs), tail, i in zip(envs, tails, ids):
        for b, t, want in zip(bufs, tail, gallery[i][1]):
            assert torch.equal(b[:P], want[:P]) and torch.equal(b[P:], t)
        assert cap.cap_set_get_position(s) == P
