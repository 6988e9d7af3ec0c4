"""Calls without the coordinate-wise test run kernels that have it compiled out (few bytes of rows per coordinate, and
read-only statistics): they must give the bits of the calls that ask for it, in every output both share."""
from __future__ import annotations

import pytest
import torch

import helpers as H
from paper_2412_21124_amd import binding as B
from paper_2412_21124_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STATS, ADAMW, GBAR = B.NT_DO_STATS, B.NT_DO_ADAMW, B.NT_WRITE_GBAR


def _step(captured, grads, state, hy, **kw):
    """Result of a step; captured: with the kernels that leave the sums to a second one, which a few tiles take in a graph only (their
    own-result kernels always have the test)."""
    if not captured:
        return B.read_result(B.normtest_step(grads, *state, hy, **kw)).as_dict()
    ws = torch.empty(B.normtest_workspace_bytes(grads.shape[0], grads.shape[1]), dtype=torch.uint8, device=DEV)
    res = torch.empty(B.RESULT_BYTES, dtype=torch.uint8, device=DEV)
    H.captured(lambda: B.normtest_step(grads, *state, hy, workspace=ws, result=res, **kw))
    return B.read_result(res).as_dict()


# both sides of the 8 bytes per coordinate, and overlapped sweeps of 64 bytes (8 bf16 / 4 fp32 rows); short and long
# statistics vectors (2^21), more and (captured) fewer tiles than end in one launch, each with a part tile
@pytest.mark.parametrize("J,gdtype", [(2, torch.bfloat16), (4, torch.bfloat16), (5, torch.bfloat16), (8, torch.bfloat16),
                                      (2, torch.float32), (3, torch.float32), (4, torch.float32), (16, torch.bfloat16)])
@pytest.mark.parametrize("flags", [STATS | ADAMW, STATS, STATS | GBAR])
@pytest.mark.parametrize("d,captured", [(4097, False), (4097, True), (3 * 16384 + 5, True), ((1 << 20) + 4099, False), ((1 << 21) + 4099, False)])
def test_same_bits_with_and_without_the_coordinate_test(J, gdtype, flags, d, captured):
    wl = synth.make("t", J, d, gdtype=gdtype, sigma=1e-2, seed=J + d, device=DEV, hyper=synth.Hyper(b_k=64, round_to=J))
    h = wl.hyper
    got = []
    for extra in (0, B.NT_COORD_TEST):
        hy = B.make_hyper(lr=h.lr, beta1=h.beta1, beta2=h.beta2, eps=h.eps, weight_decay=h.weight_decay, eta=h.eta,
                          step=h.step, b_k=h.b_k, b_max=h.b_max, round_to=h.round_to, ddof=h.ddof, flags=flags | extra)
        state = [wl.w.clone(), wl.m.clone(), wl.v.clone(), torch.zeros_like(wl.w)]
        got.append((_step(captured, wl.grads, state[:3], hy, gbar_out=state[3]), state))
    (plain, s0), (coord, s1) = got
    assert plain["coord_fail"] == -1 and coord["coord_fail"] >= 0
    for k in plain:
        if k not in ("coord_fail", "coord_max_ratio"):
            assert plain[k] == coord[k], k
    assert all(torch.equal(a, b) for a, b in zip(s0, s1))
    H.assert_stats_close(plain, H.oracle_full(wl.grads, d, J, h))


# statistics with more bytes of rows run without the test up to 2^22 coordinates of the call (16 bytes per coordinate, 8 bf16
# or 4 fp32 rows: up to 2^25); read-only ones of 15 rows, and of 11 fp32 rows, hold their loads together
@pytest.mark.parametrize("J,gdtype,edge", [(9, torch.bfloat16, 1 << 22), (13, torch.bfloat16, 1 << 22), (15, torch.bfloat16, 1 << 22),
                                           (5, torch.float32, 1 << 22), (11, torch.float32, 1 << 22), (15, torch.float32, 1 << 22),
                                           (8, torch.bfloat16, 1 << 25), (4, torch.float32, 1 << 25)])
def test_same_bits_on_both_sides_of_a_length(J, gdtype, edge):
    for d, captured in ((5, False), (8192 + 3, True), ((1 << 20) + 4099, False), (edge, False), (edge + 1, False)):
        wl = synth.make("t", J, d, gdtype=gdtype, sigma=1e-2, seed=J + d, device=DEV, hyper=synth.Hyper(b_k=64, round_to=J))
        h = wl.hyper
        for flags in (STATS, STATS | GBAR):
            got = []
            for extra in (0, B.NT_COORD_TEST):
                hy = B.make_hyper(eta=h.eta, step=h.step, b_k=h.b_k, b_max=h.b_max, round_to=h.round_to, ddof=h.ddof,
                                  flags=flags | extra)
                gbar = torch.zeros(d, dtype=torch.float32, device=DEV)
                got.append((_step(captured, wl.grads, (None, None, None), hy, d=d, gbar_out=gbar), gbar))
            (plain, g0), (coord, g1) = got
            assert plain["coord_fail"] == -1 and coord["coord_fail"] >= 0
            for k in plain:
                if k not in ("coord_fail", "coord_max_ratio"):
                    assert plain[k] == coord[k], (k, d, flags)
            assert torch.equal(g0, g1)
        if J * d <= 1 << 26:
            H.assert_stats_close(plain, H.oracle_full(wl.grads, d, J, h))
