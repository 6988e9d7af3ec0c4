"""Ragged ends and element-aligned buffers: the last tile of a vector holds whole groups of four coordinates, one group
of one to three, and nothing behind it; rows and state may start at any element.  Sizes sit around the edges of a group,
of a sweep and of a tile: tables in the classes of short vectors, matrices in those of long ones too.  Results are compared
with the oracle, and the words in front of and behind every buffer must stay what they were."""
from __future__ import annotations

import pytest
import torch

import helpers as H
from paper_2412_21124_amd import binding as B
from paper_2412_21124_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STATS, ADAMW = B.NT_DO_STATS, B.NT_DO_ADAMW

# (J, dtype): fused and statistics classes up to 16 rows; one, two and more chunks of 16 rows beyond
ROWS = [(2, torch.bfloat16), (5, torch.float32), (16, torch.bfloat16), (17, torch.float32), (40, torch.bfloat16)]
# below and at one group, a sweep of 256 and 512 threads, tiles of 2048 and 4096 coordinates, several tiles, with 1..3 over
SIZES = [1, 2, 3, 4, 1023, 1026, 2049, 4097, 6147, 16386, 20481]


def _padded(n, dtype, off, fill):
    """A buffer of n elements that starts `off` elements behind a 16-byte boundary, between guard words."""
    base = torch.full((16 + off + n + 16,), fill, dtype=dtype, device=DEV)
    return base, base[16 + off:16 + off + n]


def _guards_untouched(base, view, fill):
    lo = (view.data_ptr() - base.data_ptr()) // base.element_size()
    return bool((base[:lo] == fill).all()) and bool((base[lo + view.numel():] == fill).all())


@pytest.mark.parametrize("flags", [STATS | ADAMW | B.NT_WRITE_GBAR, STATS, STATS | B.NT_WRITE_GBAR, ADAMW])
@pytest.mark.parametrize("J,gdtype", ROWS)
def test_ragged_ends_at_every_alignment(J, gdtype, flags):
    for d in SIZES:
        wl = synth.make("t", J, d, gdtype=gdtype, sigma=1e-2, seed=17 * J + d, device=DEV,
                        hyper=synth.Hyper(b_k=64, round_to=J, step=3))
        h = wl.hyper
        # every row at an offset of its own, NaN around it: a value from outside would show in every result
        rows = [_padded(d, gdtype, j % 8, float("nan"))[1] for j in range(J)]
        for r, g in zip(rows, wl.grads):
            r.copy_(g)
        state = [_padded(d, torch.float32, k + 1, 5.0) for k in range(4)]
        for (_, s), src in zip(state, (wl.w, wl.m, wl.v)):
            s.copy_(src)
        w, m, v, gbar = (s for _, s in state)
        hy = B.make_hyper(lr=h.lr, beta1=h.beta1, beta2=h.beta2, eps=h.eps, weight_decay=h.weight_decay, eta=h.eta,
                          step=h.step, b_k=h.b_k, b_max=h.b_max, round_to=h.round_to, ddof=h.ddof, flags=flags)
        res = B.read_result(B.normtest_step_rows(rows, w, m, v, hy, gbar_out=gbar)).as_dict()
        if flags & STATS:
            ref = H.oracle_full(wl.grads, d, J, h)
            H.assert_stats_close(res, ref)
        if flags & ADAMW:
            H.oracle_adamw_check(wl.grads, d, wl.w, wl.m, wl.v, w, m, v, h)
        else:
            assert torch.equal(w, wl.w) and torch.equal(m, wl.m) and torch.equal(v, wl.v)
        if flags & B.NT_WRITE_GBAR:
            # the mean is the fp64 row sum, scaled and rounded once: half an ulp, and one more for the scaling
            ref_gbar = wl.grads.double().mean(0)
            assert bool(((gbar.double() - ref_gbar).abs() <= 2.0 ** -23 * ref_gbar.abs() + 1e-45).all())
        for base, s in state:
            assert _guards_untouched(base, s, 5.0), (d, "guard words")


# with `whole` the vector is the start of a long one: deferred updates (16 bf16 and 8 fp32 rows), the shapes beyond 16 and 20
# rows, with (24) and without (40) a copy of their walk for whole tiles, and statistics in 16384-coordinate tiles
@pytest.mark.parametrize("whole", [None, 1 << 26])
@pytest.mark.parametrize("flags", [STATS | ADAMW | B.NT_WRITE_GBAR, STATS, STATS | B.NT_WRITE_GBAR, ADAMW])
@pytest.mark.parametrize("J,gdtype", [(3, torch.bfloat16), (16, torch.bfloat16), (8, torch.float32), (17, torch.bfloat16),
                                      (20, torch.float32), (24, torch.bfloat16), (40, torch.bfloat16), (40, torch.float32)])
def test_ragged_ends_of_a_matrix(J, gdtype, flags, whole):
    """The same of one matrix with an odd row stride and NaN between its rows, around the edges of the 8192- and
    16384-coordinate tiles too; and the same bits as from a table of the same rows."""
    kw = {} if whole is None else {"shard": B.nt_shard_info(0, 1, 0, whole)}
    for d in (1, 2, 3, 4, 1026, 2049, 4099, 8191, 8194, 16387):
        wl = synth.make("t", J, d, gdtype=gdtype, sigma=1e-2, seed=J + d, device=DEV,
                        hyper=synth.Hyper(b_k=64, round_to=J, step=3))
        h = wl.hyper
        hy = B.make_hyper(lr=h.lr, beta1=h.beta1, beta2=h.beta2, eps=h.eps, weight_decay=h.weight_decay, eta=h.eta,
                          step=h.step, b_k=h.b_k, b_max=h.b_max, round_to=h.round_to, ddof=h.ddof, flags=flags)
        big = torch.full((J, d + 5 + d % 2), float("nan"), dtype=gdtype, device=DEV)
        view = big[:, 3:3 + d]
        view.copy_(wl.grads[:, :d])
        got = []
        for table in (False, True):
            state = [_padded(d, torch.float32, k + 1, 5.0) for k in range(4)]
            for (_, s), src in zip(state, (wl.w, wl.m, wl.v)):
                s.copy_(src)
            w, m, v, gbar = (s for _, s in state)
            if table:
                res = B.normtest_step_rows([view[j] for j in range(J)], w, m, v, hy, gbar_out=gbar, **kw)
            else:
                res = B.normtest_step(view, w, m, v, hy, d=d, gbar_out=gbar, **kw)
            got.append((B.read_result(res).as_dict(), state))
            for base, s in state:
                assert _guards_untouched(base, s, 5.0), (d, "guard words")
        (res, state), (other, other_state) = got
        if flags & STATS:
            assert res == other
            H.assert_stats_close(res, H.oracle_full(wl.grads, d, J, h))
        for (_, a), (_, b) in zip(state, other_state):
            assert torch.equal(a, b)
        if flags & ADAMW and d > 4:
            # (of one to four coordinates one may be a moment that cancels: its error is then half an ulp of the summands, which
            # the root mean square of so few does not cover; they have the table's bits)
            H.oracle_adamw_check(wl.grads, d, wl.w, wl.m, wl.v, *(s for _, s in state[:3]), h)
        if flags & B.NT_WRITE_GBAR:
            # as above: half an ulp, and one more for the scaling
            ref_gbar = wl.grads[:, :d].double().mean(0)
            assert bool(((state[3][1].double() - ref_gbar).abs() <= 2.0 ** -23 * ref_gbar.abs() + 1e-45).all())
