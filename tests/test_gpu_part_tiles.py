"""A vector that ends inside a tile against the same vector continued with zeros to the tile's end: its last group of four
coordinates is loaded from another place (and moved, where there are sums), and every output has to have the bits of the whole tile."""
from __future__ import annotations

import pytest
import torch

from paper_2412_21124_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STATS, ADAMW, GBAR, COORD = B.NT_DO_STATS, B.NT_DO_ADAMW, B.NT_WRITE_GBAR, B.NT_COORD_TEST
# fewer coordinates than one load, one load, and 1 to 3 past the end of a sweep or tile, where the group's load starts before it
SIZES = [1, 3, 4, 5, 511, 513, 1026, 2049, 4098, 6147, 8193, 16387, 20482]
HYPER = dict(lr=3e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1, step=5, b_k=64, b_max=8192, round_to=8)


def _step(rows, state, d, flags, shard, table):
    w, m, v, gbar = (s[:d].contiguous() for s in state)
    hy = B.make_hyper(**HYPER, flags=flags)
    if table:
        res = B.normtest_step_rows([r[:d].contiguous() for r in rows], w, m, v, hy, gbar_out=gbar, shard=shard)
    else:
        res = B.normtest_step(rows[:, :d].contiguous(), w, m, v, hy, gbar_out=gbar, shard=shard)
    return B.read_result(res).as_dict(), (w, m, v, gbar)


# the classes of short vectors, of a part of a longer one, and of a part of a long one
@pytest.mark.parametrize("whole", [None, 1 << 22, 1 << 26])
@pytest.mark.parametrize("flags", [STATS | ADAMW | GBAR, STATS | COORD, STATS | GBAR, ADAMW, ADAMW | GBAR])
@pytest.mark.parametrize("J,gdtype,table", [(4, torch.bfloat16, False), (5, torch.float32, True), (16, torch.bfloat16, True),
                                            (16, torch.float32, False), (19, torch.float32, False), (18, torch.bfloat16, True), (24, torch.bfloat16, True),
                                            (47, torch.bfloat16, False), (33, torch.float32, True)])
def test_bits_of_the_vector_continued_with_zeros(J, gdtype, table, flags, whole):
    n = 32768
    g = torch.Generator(device=DEV).manual_seed(J)
    full = (torch.randn(J, n, generator=g, device=DEV) * 1e-2).to(gdtype)
    state = [torch.rand(n, generator=g, device=DEV) * 0.02 for _ in range(4)]
    shard = None if whole is None else B.nt_shard_info(0, 8, 0, whole)
    for d in SIZES:
        rows, st = full.clone(), [s.clone() for s in state]
        rows[:, d:] = 0
        for s in st:
            s[d:] = 0
        end = (d + 16383) // 16384 * 16384   # every tile size divides this
        # more tiles, all of zeros, add zeros: the sums keep their bits too
        got, a = _step(rows, st, d, flags, shard, table)
        want, b = _step(rows, st, end, flags, shard, table)
        for x, y in zip(a[:3] if not flags & GBAR else a, b):
            assert torch.equal(x, y[:d]), d
        if flags & STATS:
            for k in ("A", "B", "C", "A_lo", "B_lo", "C_lo", "T", "coord_fail", "coord_max_ratio"):
                assert got[k] == want[k], (d, k)


def test_adamw_from_a_mean_continued_with_zeros():
    n = 32768
    vec = [torch.rand(n, device=DEV) * 0.02 for _ in range(4)]
    hy = B.make_hyper(**HYPER)
    for d in SIZES:
        st = [torch.cat([s[:d], torch.zeros(n - d, device=DEV)]) for s in vec]
        outs = []
        for k in (d, n):
            gbar, w, m, v = (s[:k].contiguous() for s in st)
            B.normtest_adamw_gbar(gbar, w, m, v, hy, 0.5)
            outs.append((w, m, v))
        for x, y in zip(*outs):
            assert torch.equal(x, y[:d]), d


# how many blocks a CU holds, and launches of another length: the first coordinates of a longer vector, on both sides of each edge
@pytest.mark.parametrize("J,flags,edge", [(8, ADAMW, 1 << 23), (8, STATS | ADAMW, 1 << 25), (2, ADAMW, 1 << 28),
                                          (5, STATS | GBAR, 1 << 25), (9, STATS | GBAR, 1 << 25)])
def test_state_does_not_depend_on_the_length(J, flags, edge):
    rows = (torch.randn(J, edge + 4099, device=DEV) * 1e-2).to(torch.bfloat16)
    state = [torch.rand(edge + 4099, device=DEV) * 0.02 for _ in range(4 if flags & GBAR else 3)]
    outs = []
    for d in (edge - 4096 + 1, edge + 4099):
        st = [s[:d].clone() for s in state]
        B.normtest_step(rows, *st[:3], B.make_hyper(**HYPER, flags=flags), d=d, gbar_out=st[3] if flags & GBAR else None)
        outs.append(st)
    for x, y in zip(*outs):
        assert torch.equal(x, y[:x.numel()])
