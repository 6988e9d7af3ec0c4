"""Steps whose own kernel writes the result: vectors of one tile or a few, and AdamW only at any length.  Result and workspace start
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


# one tile is 4096 coordinates up to 16 rows and 2048 beyond; with one more coordinate the last block adds up the partials
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


def _same(a, b):
    assert a.keys() == b.keys()
    for k in a:
        assert a[k] == b[k] or (a[k] != a[k] and b[k] != b[k]), (k, a[k], b[k])


# a tile, whose partial is the total; one coordinate more, which ends at the counter, and under capture in the reduction kernel
@pytest.mark.parametrize("J,gdtype,tile", [(2, torch.float32, 4096), (16, torch.bfloat16, 4096), (33, torch.float32, 2048)])
@pytest.mark.parametrize("value", [math.inf, 1e20])   # in one row; in all rows, finite, where only the squares overflow
def test_sums_that_are_not_finite_read_the_same_on_every_way(J, gdtype, tile, value):
    wl = synth.make("t", J, tile + 1, gdtype=gdtype, sigma=1e-2, seed=J, device=DEV, hyper=synth.Hyper(b_k=64, round_to=J))
    wl.grads[:1 if math.isinf(value) else J, 7] = value
    h = wl.hyper
    hy = B.make_hyper(lr=h.lr, beta1=h.beta1, beta2=h.beta2, eps=h.eps, weight_decay=h.weight_decay, eta=h.eta,
                      step=h.step, b_k=h.b_k, b_max=h.b_max, round_to=h.round_to, ddof=h.ddof)
    gbar = torch.empty(tile + 1, dtype=torch.float32, device=DEV)
    ws = torch.empty(B.normtest_workspace_bytes(J, tile + 1), dtype=torch.uint8, device=DEV)

    def captured(d, s):
        out = torch.empty(B.RESULT_BYTES, dtype=torch.uint8, device=DEV)
        H.captured(lambda: B.normtest_step(wl.grads, *s, hy, d=d, workspace=ws, result=out))
        return out

    ways = {"matrix": lambda d, s: B.normtest_step(wl.grads, *s, hy, d=d),
            "table": lambda d, s: B.normtest_step_rows(list(wl.grads), *s, hy, d=d),
            "static": lambda d, s: B.normtest_step_static(
                wl.grads, *s, hy, torch.empty(B.RESULT_BYTES, dtype=torch.uint8, device=DEV), d=d),
            "clipped": lambda d, s: B.normtest_step_clipped(wl.grads, *s, gbar, 1.0, hy, d=d),
            "captured": captured}
    got = {}
    for name, way in ways.items():
        for d in (tile, tile + 1):
            state = [t.clone() for t in (wl.w, wl.m, wl.v)]
            res = B.read_result(way(d, state)).as_dict()
            assert res["status"] == B.NT_STATUS_NONFINITE and res["pass"] == 1 and res["next_b"] == h.b_k
            # the double-double sums turn an infinite partial into NaN; a norm that is not a number clips nothing
            for k in ("A", "B", "gbar_sq", "T"):
                assert math.isnan(res[k]), (name, d, k, res[k])
            assert res["clip_coef"] == 1.0
            got[name, d] = res, state
    for d in (tile, tile + 1):
        res, state = got["matrix", d]
        for name in ways:
            _same(res, got[name, d][0])
            for a, b in zip(state, got[name, d][1]):
                assert torch.allclose(a[:d], b[:d], rtol=0.0, atol=0.0, equal_nan=True), (name, d)


@pytest.mark.parametrize("J,d", [(2, 3 * (1 << 25) + 5), (10, (1 << 26) + 3), (20, 5 * (1 << 23) + 3)])
def test_adamw_only_writes_its_result_in_the_last_launch(J, d):
    """The record goes into memory of row 0 that a launch between the first and the last reads: had it been written before,
    that launch would average its words.  Every launch class of AdamW only that is walked in several launches."""
    wl = synth.make("t", J, d, gdtype=torch.bfloat16, sigma=1e-2, seed=5, device=DEV, hyper=synth.Hyper(b_k=96, round_to=J))
    h = wl.hyper
    hy = B.make_hyper(lr=h.lr, beta1=h.beta1, beta2=h.beta2, eps=h.eps, weight_decay=h.weight_decay, eta=h.eta,
                      step=h.step, b_k=h.b_k, b_max=h.b_max, round_to=h.round_to, ddof=h.ddof, flags=ADAMW)
    want = [t.clone() for t in (wl.w, wl.m, wl.v)]
    B.normtest_step(wl.grads, *want, hy)
    at = d // 2 // 64 * 64
    result = wl.grads[0, at:at + B.RESULT_BYTES // 2].view(torch.uint8)
    res = B.read_result(B.normtest_step(wl.grads, wl.w, wl.m, wl.v, hy, result=result)).as_dict()
    assert res["status"] == B.NT_STATUS_NO_STATS and res["pass"] == 1 and res["next_b"] == 96
    for a, b in zip(want, (wl.w, wl.m, wl.v)):
        assert torch.equal(a, b)


# every row count with a kernel of its own, both shapes beyond 16 rows and the one beyond 20; one tile in the classes of short
# vectors and, for a part of a long one, in those of long vectors
@pytest.mark.parametrize("whole", [None, 1 << 26])
@pytest.mark.parametrize("gdtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("flags", [STATS | ADAMW, STATS, STATS | GBAR, STATS | COORD, ADAMW])
def test_every_class_leaves_a_result(gdtype, flags, whole):
    """Whether the step's own kernel writes the result or a second one does, it is written, and it is the one that the same
    rows give in a pointer table and, continued with zeros into a second tile and captured, by way of the reduction kernel."""
    d, longer = 700, 16384 + 700
    for J in [*range(2, 22), 33]:
        wl = synth.make("t", J, d, gdtype=gdtype, sigma=1e-2, seed=J, device=DEV, hyper=synth.Hyper(b_k=64, round_to=J))
        kw = {} if whole is None else {"shard": B.nt_shard_info(0, 1, 0, whole)}
        w, m, v = (t.clone() for t in (wl.w, wl.m, wl.v))
        res, _ = _run(wl, flags, **kw)
        h = wl.hyper
        hy = B.make_hyper(lr=h.lr, beta1=h.beta1, beta2=h.beta2, eps=h.eps, weight_decay=h.weight_decay, eta=h.eta,
                          step=h.step, b_k=h.b_k, b_max=h.b_max, round_to=h.round_to, ddof=h.ddof, flags=flags)
        gbar = torch.empty(d, dtype=torch.float32, device=DEV)
        out = torch.full((B.RESULT_BYTES,), 0xA5, dtype=torch.uint8, device=DEV)
        _same(res, B.read_result(B.normtest_step_rows(list(wl.grads), w, m, v, hy, gbar_out=gbar, result=out, **kw)).as_dict())
        grads = torch.zeros(J, longer, dtype=gdtype, device=DEV)
        grads[:, :d] = wl.grads[:, :d]
        state = [torch.zeros(longer, dtype=torch.float32, device=DEV) for _ in range(4)]
        ws = torch.empty(B.normtest_workspace_bytes(J, longer), dtype=torch.uint8, device=DEV)
        out.fill_(0xA5)
        H.captured(lambda: B.normtest_step(grads, *state[:3], hy, gbar_out=state[3], workspace=ws, result=out, **kw))
        _same(res, B.read_result(out).as_dict())
        assert (res["status"] == B.NT_STATUS_NO_STATS) == (not flags & STATS)
        for a, b in zip((w, m, v), (wl.w, wl.m, wl.v)):
            assert torch.equal(a, b)
