"""Ends of segments around every tile size, bit for bit against the oracle.

A tile is 64 lanes x 1-4 slots x 16 bytes of each member stream; a segment's
last tile holds fewer whole vectors and up to N - 1 single elements (N = 4
fp32, 8 bf16).  Sizes step over each of those edges: in small launches, which
take one slot per lane for every unit, and in larger ones, where units of up
to three members take two or four.  Every buffer lies between guard bytes that
must not change, and one member of each group does not update.
"""
import os
import re

import numpy as np
import pytest

from oracle import preduce as op
from seedgen import f32_to_bf16_bits

from gpu_util import compare, log

pytestmark = pytest.mark.gpu

GUARD = 512  # bytes before and after every segment

HERE = os.path.dirname(os.path.abspath(__file__))
POLICY = os.path.join(HERE, "..", "paper_1909_08029_amd", "csrc", "rip_launch_policy.h")


def _one_slot_work():
    """Most one-slot tiles of a launch that takes one slot for every unit."""
    with open(POLICY) as f:
        return int(re.search(r"kOneSlotWork = (\d+);", f.read()).group(1))


def _arrays(rng, n, sizes, bf16):
    out = [(rng.standard_normal((n, m)) * 0.5).astype(np.float32) for m in sizes]
    return [f32_to_bf16_bits(x) for x in out] if bf16 else out


class Guarded:
    """n replicas of the segments in one buffer, GUARD bytes around each."""

    def __init__(self, arrays):
        import torch
        esize = arrays[0].dtype.itemsize
        self.dtype, self.n = arrays[0].dtype, arrays[0].shape[0]
        self.spans, at = [], GUARD
        for r in range(self.n):
            row = []
            for x in arrays:
                row.append((at, at + x.shape[1] * esize))
                at = (at + x.shape[1] * esize + GUARD + 255) // 256 * 256
            self.spans.append(row)
        host = np.random.default_rng(1).integers(0, 256, at + GUARD, dtype=np.uint8)
        for r, row in enumerate(self.spans):
            for x, (a, b) in zip(arrays, row):
                host[a:b] = x[r].view(np.uint8)
        self.before, self.dev = host, torch.from_numpy(host.copy()).cuda()
        tdt = torch.bfloat16 if esize == 2 else torch.float32
        self.views = [[self.dev[a:b].view(tdt) for a, b in row] for row in self.spans]

    def segments(self):
        """The segments now; asserts that no byte outside them changed."""
        now = self.dev.cpu().numpy()
        inside = np.zeros(now.size, bool)
        for row in self.spans:
            for a, b in row:
                inside[a:b] = True
        assert np.array_equal(now[~inside], self.before[~inside]), "bytes outside a segment changed"
        return [np.stack([now[a:b].view(self.dtype) for a, b in (row[s] for row in self.spans)])
                for s in range(len(self.spans[0]))]


def _check(bf16, mom, k, sizes, average=False, wd=0.0, nesterov=False, lone=1):
    import torch
    import paper_1909_08029_amd as rip
    rng = np.random.default_rng(1000 * k + sum(sizes))
    n = k + lone + 1                       # the last replica is left alone
    p, g, v = (_arrays(rng, n, sizes, bf16) for _ in range(3))
    P, G, V = Guarded(p), Guarded(g), Guarded(v)
    rep = rip.Replicas(P.views, G.views, V.views)
    group = [tuple(range(k))] if k > 1 else []
    active = [] if average else [i for i in range(k + lone) if i != 1 or k < 3]
    lr, mu = (None, 0.0) if average else (0.1, 0.9 if mom else 0.0)
    rip.rip_preduce(rep, group, active, lr=lr, momentum=mu, weight_decay=wd, nesterov=nesterov)
    torch.cuda.synchronize()
    dt = op.BF16 if bf16 else op.F32
    want = [op.step(p[s], g[s], v[s] if mom else None, group, active, lr or 0.0,
                    mu if mom else None, dt, True, wd, nesterov) for s in range(len(sizes))]
    what = f"bf16={bf16} mom={mom} k={k} sizes={sizes}"
    for s, (wp, wv) in enumerate(want):
        compare(P.segments()[s], wp, int(bf16), what + " param")
        compare(V.segments()[s], wv if mom else v[s], int(bf16), what + " mom")
        compare(G.segments()[s], g[s], int(bf16), what + " grad")
    rep.close()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("mom", [False, True])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 7, 8])
def test_segment_ends(bf16, mom, k):
    N = 8 if bf16 else 4
    sizes = {1, N - 1, N, N + 1, 2 * N + 3}
    for slots in (1, 2, 4):
        tile = 64 * N * slots
        sizes |= {tile - N - 1, tile - 1, tile, tile + 1, tile + N, 2 * tile + 63 * N + N - 1}
    log(f"case bf16={bf16} mom={mom} k={k}: {len(sizes)} sizes")
    for m in sorted(sizes):
        _check(bf16, mom, k, [m])
    _check(bf16, mom, k, [5, 64 * N + 1, 1, 256 * N + N + 1, 64 * N])     # separate segments
    _check(bf16, mom, k, [64 * N + 3], wd=1e-2, nesterov=mom)
    if k > 1:
        _check(bf16, False, k, [64 * N + 3, 7], average=True)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("mom", [False, True])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_segment_ends_of_several_slots(bf16, mom, k):
    """Ends in every slot of a tile of two or four slots: segments of a few
    tiles each beside one that makes the launch large enough for them, then
    flat ranges that end in each slot (for bf16 on a lone element)."""
    N = 8 if bf16 else 4
    slot, tile = 64 * N, 64 * N * 4
    units = 2                              # a group and a lone update, or two of those
    base = tile * (-(-_one_slot_work() // (4 * units)) + 1)
    edges = {1, N - 1, N, N + 1, 2 * N + 3, 2 * tile - 1, 2 * tile}
    for u in range(1, 5):
        edges |= {u * slot + d for d in (-N - 1, -N, -1, 0, 1, N - 1, N, N + 1)}
        edges |= {tile + u * slot - 1, tile + u * slot + 1}
    log(f"case slots bf16={bf16} mom={mom} k={k}: {len(edges)} segments after {base} elements")
    flat = [base + u * slot + d for u in range(4) for d in (1, 32 * N + N + 1)]
    for sizes in ([base] + sorted(edges), *([m] for m in flat)):
        assert units * sum(-(-m // slot) for m in sizes) > _one_slot_work()
        _check(bf16, mom, k, sizes)
    _check(bf16, mom, k, [base + 3 * slot + 5, 2 * slot + 1], wd=1e-2, nesterov=mom)
    if k > 1:
        _check(bf16, False, k, [base + slot + 3, 2 * slot + 7], average=True)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("mom", [False, True])
@pytest.mark.parametrize("k", [9, 16, 17, 31, 33, 64, 65, 127, 130, 254])
def test_wide_groups(bf16, mom, k):
    """Groups above eight: their members are shared by the waves of a
    workgroup, evenly and in rounds.  A lone replica beside the group runs in
    the same launch while that is small, in one of its own above."""
    import paper_1909_08029_amd as rip
    N = 8 if bf16 else 4
    log(f"case wide bf16={bf16} mom={mom} k={k}")
    for m in (1, N, N + 1, 64 * N - 1, 64 * N, 64 * N + N + 3, 3 * 64 * N + 63 * N + 1):
        _check(bf16, mom, k, [m], lone=k % 2)
        assert rip.rip_last_launch_count() == 1
    _check(bf16, mom, k, [5, 64 * N + 1, 1, 64 * N], lone=0)
    _check(bf16, mom, k, [64 * N + 3], wd=1e-2, nesterov=mom, lone=0)
    _check(bf16, False, k, [64 * N + 3, 7], average=True, lone=0)
    try:                                   # workgroups that loop over tiles, one per CU
        rip.rip_set_max_blocks(3)
        rip.rip_set_blocks_per_cu(1)
        _check(bf16, mom, k, [64 * N * 11 + N + 1, 64 * N], lone=0)
    finally:
        rip.rip_set_max_blocks(0)
        rip.rip_set_blocks_per_cu(0)
    if k < 20:
        _check(bf16, mom, k, [64 * N * 1800 + 3], lone=1)
        assert rip.rip_last_launch_count() == 2
