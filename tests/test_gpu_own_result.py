"""Steps whose own kernel writes the result: vectors of one tile, and AdamW only at any length.  Result and workspace start
as garbage; the sums, the decision and the per-layer table read from the workspace afterwards must be the oracle's."""
from __future__ import annotations

import math

import pytest
import torch

import helpers as H
from paper_2412_21124_amd import binding as B
from paper_2412_21124_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STATS, ADAMW, GBAR, COORD, PARTIAL = (B.NT_DO_STATS, B.NT_DO_ADAMW, B.NT_WRITE_GBAR, B.NT_COORD_TEST, B.NT_PARTIAL)


def _run(wl, flags, **kw):
    h = wl.hyper
    hy = B.make_hyper(lr=h.lr, beta1=h.beta1, beta2=h.beta2, eps=h.eps, weight_decay=h.weight_decay, eta=h.eta,
                      step=h.step, b_k=h.b_k, b_max=h.b_max, round_to=h.round_to, ddof=h.ddof, flags=flags)
    ws = torch.full((B.normtest_workspace_bytes(wl.J, wl.d),), 0xA5, dtype=torch.uint8, device=DEV)
    res = torch.full((B.RESULT_BYTES,), 0xA5, dtype=torch.uint8, device=DEV)
    gbar = torch.empty(wl.d, dtype=torch.float32, device=DEV)
    B.normtest_step(wl.grads, wl.w, wl.m, wl.v, hy, gbar_out=gbar, workspace=ws, result=res, **kw)
    return B.read_result(res).as_dict(), ws


# one tile is 4096 coordinates up to 16 rows and 2048 beyond; one more coordinate takes the two-kernel way
@pytest.mark.parametrize("J,gdtype,tile", [(2, torch.bfloat16, 4096), (16, torch.float32, 4096), (33, torch.bfloat16, 2048)])
@pytest.mark.parametrize("flags", [STATS | ADAMW, STATS, STATS | GBAR, STATS | ADAMW | COORD, STATS | ADAMW | PARTIAL])
def test_one_tile(J, gdtype, tile, flags):
    for d in (1, tile - 1, tile, tile + 1):
        wl = synth.make("t", J, d, gdtype=gdtype, sigma=1e-2, seed=J + d, device=DEV, hyper=synth.Hyper(b_k=64, round_to=J))
        ref = H.oracle_full(wl.grads, d, J, wl.hyper)
        res, ws = _run(wl, flags)
        H.assert_stats_close(res, ref, partial=bool(flags & PARTIAL))
        if not flags & PARTIAL:
            H.assert_decision_matches(res, ref, wl.hyper)
        assert (res["coord_fail"] >= 0) == bool(flags & COORD)
        layers = B.read_layers(B.normtest_layer_stats(
            wl.grads, torch.tensor([0, d], dtype=torch.int64, device=DEV), ws))
        assert layers[0].n == d
        # the table adds a part tile coordinate by coordinate in fp64, the step in fp32 groups of four: two roundings
        for k in ("A", "B", "C"):
            assert abs(getattr(layers[0], k) - res[k]) <= 2 * 2.0 ** -24 * res[k], k


@pytest.mark.parametrize("J,gdtype,d", [(3, torch.bfloat16, 5), (8, torch.float32, 70_001), (40, torch.bfloat16, 9000),
                                        (10, torch.bfloat16, (1 << 26) + 3)])   # the last: several launches, deferred update
def test_adamw_only_reports_no_statistics(J, gdtype, d):
    wl = synth.make("t", J, d, gdtype=gdtype, sigma=1e-2, seed=3, device=DEV, hyper=synth.Hyper(b_k=96, round_to=J))
    res, ws = _run(wl, ADAMW)
    assert res["status"] == B.NT_STATUS_NO_STATS and res["pass"] == 1 and res["next_b"] == 96
    assert res["clip_coef"] == 1.0 and res["coord_fail"] == -1 and res["coord_max_ratio"] == -1.0
    assert all(math.isnan(res[k]) for k in ("A", "B", "C", "A_lo", "B_lo", "C_lo", "gbar_sq", "var_l1", "T"))
    layers = B.read_layers(B.normtest_layer_stats(wl.grads, torch.tensor([0, d], dtype=torch.int64, device=DEV), ws))
    assert layers[0].status & B.NT_STATUS_NO_STATS
