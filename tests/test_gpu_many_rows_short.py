"""More than 16 rows on both sides of the lengths at which the shape of the blocks changes: the same bits in the state and the
stored mean, and the sums of the oracle."""
from __future__ import annotations

import pytest
import torch

import helpers as H
from paper_2412_21124_amd import binding as B
from paper_2412_21124_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STATS, ADAMW, GBAR = B.NT_DO_STATS, B.NT_DO_ADAMW, B.NT_WRITE_GBAR


@pytest.mark.parametrize("J,gdtype,edge", [(17, torch.bfloat16, 1 << 20), (32, torch.bfloat16, 1 << 20), (33, torch.bfloat16, 1 << 19),
                                           (20, torch.float32, 1 << 19), (48, torch.float32, 1 << 19)])
@pytest.mark.parametrize("flags", [STATS | ADAMW | GBAR, STATS, ADAMW])
def test_same_outputs_on_both_sides_of_a_length(J, gdtype, edge, flags):
    if flags == ADAMW:
        edge = 1 << 19
    wl = synth.make("t", J, edge + 1, gdtype=gdtype, sigma=1e-2, seed=J, device=DEV, hyper=synth.Hyper(b_k=64, round_to=J))
    h = wl.hyper
    hy = B.make_hyper(lr=h.lr, beta1=h.beta1, beta2=h.beta2, eps=h.eps, weight_decay=h.weight_decay, eta=h.eta, step=h.step,
                      b_k=h.b_k, b_max=h.b_max, round_to=h.round_to, ddof=h.ddof, flags=flags)
    outs = []
    for d in (edge, edge + 1):
        state = [t.clone() for t in (wl.w, wl.m, wl.v)] + [torch.zeros(edge + 1, device=DEV)]
        res = B.read_result(B.normtest_step(wl.grads, *state[:3], hy, d=d, gbar_out=state[3])).as_dict()
        if flags & STATS:
            H.assert_stats_close(res, H.oracle_full(wl.grads, d, J, h))
        outs.append(state)
    for a, b in zip(*outs):
        assert torch.equal(a[:edge], b[:edge])


# just past a generation of blocks, and where the class for long vectors takes over again; one more coordinate, of zeros, on
# the other side of the edge adds nothing
@pytest.mark.parametrize("J,gdtype,edge", [(33, torch.bfloat16, (1 << 23) * 13 // 16 - 1), (33, torch.bfloat16, 1 << 23),
                                           (40, torch.bfloat16, (1 << 23) * 11 // 8), (33, torch.float32, (1 << 23) * 5 // 4),
                                           (21, torch.bfloat16, 1 << 24), (24, torch.bfloat16, (1 << 23) * 9 // 4),
                                           (33, torch.bfloat16, (1 << 23) * 17 // 8), (20, torch.float32, (1 << 24) - 1),
                                           (48, torch.bfloat16, (1 << 23) * 3 // 4 - 1), (33, torch.float32, (1 << 23) * 9 // 8),
                                           (64, torch.bfloat16, (1 << 23) * 21 // 16), (33, torch.float32, (1 << 23) * 17 // 16)])
@pytest.mark.parametrize("flags", [STATS | ADAMW, STATS | GBAR, ADAMW])
def test_same_outputs_in_generations_and_in_short_tiles(J, gdtype, edge, flags):
    g = torch.Generator(device=DEV).manual_seed(J)
    rows = torch.empty((J, edge + 1), dtype=gdtype, device=DEV)
    for r in rows:
        r.copy_(torch.randn(edge + 1, generator=g, device=DEV) * 1e-2)
    rows[:, edge] = 0
    start = [torch.rand(edge + 1, generator=g, device=DEV) * 0.02 for _ in range(4)]
    hy = B.make_hyper(lr=4e-4, step=10, b_k=256, b_max=8192, round_to=J, flags=flags)
    outs, sums = [], []
    for d in (edge, edge + 1):
        state = [t.clone() for t in start]
        sums.append(B.read_result(B.normtest_step(rows, *state[:3], hy, d=d, gbar_out=state[3])).as_dict())
        outs.append(state)
    for a, b in zip(*outs):
        assert torch.equal(a[:edge], b[:edge])
    for k in ("A", "B", "C") if flags & STATS else ():   # fp32 terms of four coordinates, the same ones, added in fp64 in another order
        assert sums[0][k] == pytest.approx(sums[1][k], rel=1e-13)
