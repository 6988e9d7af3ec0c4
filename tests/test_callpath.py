"""The native call path of the binding against its checks in Python: what it takes gives the same outputs, what it does not take is
refused or accepted as without it."""
from __future__ import annotations

import threading

import pytest
import torch

from paper_2412_21124_amd import binding as B

FULL = B.NT_DO_STATS | B.NT_DO_ADAMW


def _outcome(call):
    try:
        return call()
    except Exception as e:   # any: the type and the words are compared
        return type(e), str(e)


def _both(monkeypatch, call):
    B.lib()
    with_it = _outcome(call)
    with monkeypatch.context() as m:
        m.setattr(B, "_fast", None)
        return with_it, _outcome(call)


# without a GPU nothing is taken, and every call ends as it does in Python
def test_host_tensors_are_refused(monkeypatch):
    g, v = torch.zeros(3, 64), torch.zeros(64)
    ws, res, hy = torch.zeros(4096, dtype=torch.uint8), torch.zeros(B.RESULT_BYTES, dtype=torch.uint8), B.make_hyper(flags=FULL)
    kw = dict(workspace=ws, result=res)
    calls = [lambda: B.normtest_step(g, v, v, v, hy, **kw), lambda: B.normtest_step(g.numpy(), v, v, v, hy, **kw),
             lambda: B.normtest_step(None, v, v, v, hy, **kw), lambda: B.normtest_step_rows(list(g), v, v, v, hy, table=v, **kw),
             lambda: B.normtest_step_rows([], v, v, v, hy, table=v, **kw), lambda: B.normtest_step_clipped(g, v, v, v, v, 1.0, hy, **kw),
             lambda: B.normtest_adamw_gbar(v, v, v, v, hy)]
    for call in calls:
        a, b = _both(monkeypatch, call)
        assert a == b and isinstance(a[0], type)
    L = B.lib()
    assert B._fast.step(L.normtest_step_entry, g, v, v, v, hy, None, None, None, ws, res) is None
    assert B._fast.step(0, g, v, v, v, hy, None, None, None, ws, res) is None
    with pytest.raises(TypeError):
        B._fast.step(L.normtest_step_entry, g)


class _Recorded:
    """The native call path, and what it has returned: None for a call that it left to Python."""
    def __init__(self, fast):
        self.fast, self.back = fast, []

    def __getattr__(self, name):
        def call(*args):
            self.back.append(getattr(self.fast, name)(*args))
            return self.back[-1]
        return call


class _Gpu:
    def __init__(self, gdtype=torch.bfloat16, J=5, d=3001, ld=3008):
        g = torch.Generator(device="cuda").manual_seed(3)
        self.grads = (torch.randn(J, ld, generator=g, device="cuda") * 1e-2).to(gdtype)
        self.state = [torch.rand(d, generator=g, device="cuda") * 0.02 for _ in range(3)]
        self.gbar = torch.zeros(d, device="cuda")
        self.ws = torch.empty(B.normtest_workspace_bytes(J, ld), dtype=torch.uint8, device="cuda")
        self.res = torch.zeros(B.RESULT_BYTES, dtype=torch.uint8, device="cuda")
        self.kw = dict(workspace=self.ws, result=self.res)
        self.d = d

    def run(self, call):
        """What the call returns or raises, and every output's bits."""
        s = [t.clone() for t in self.state]
        self.gbar.zero_()
        self.res.zero_()
        back = _outcome(lambda: call(*s))
        torch.cuda.synchronize()
        return ("result" if back is self.res else back), [t.clone() for t in (*s, self.gbar, self.res)]

    def same(self, monkeypatch, call, taken, accepted=True):
        """The call ends as it does in Python.  taken: the native call path has made it, and nobody else."""
        B.lib()
        with monkeypatch.context() as m:
            seen = _Recorded(B._fast)
            m.setattr(B, "_fast", seen)
            a = self.run(call)
            m.setattr(B, "_fast", None)
            b = self.run(call)
        assert a[0] == b[0]
        assert all(torch.equal(x, y) for x, y in zip(a[1], b[1]))
        assert (a[0] in ("result", None)) == accepted, a[0]
        if accepted:
            assert (seen.back == [B.NT_OK]) if taken else (seen.back in ([], [None])), seen.back


@pytest.mark.gpu
@pytest.mark.parametrize("gdtype", [torch.bfloat16, torch.float32])
def test_outputs_are_those_of_the_python_path(monkeypatch, gdtype):
    c = _Gpu(gdtype)
    g, d = c.grads, c.d
    hy, stats = B.make_hyper(step=4, flags=FULL | B.NT_WRITE_GBAR), B.make_hyper(flags=B.NT_DO_STATS)
    shard = B.nt_shard_info(1, 4, d, 4 * d)
    rows = [r[:d].clone() for r in g]
    table = B.make_row_table(rows)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step(g, w, m, v, hy, d=d, gbar_out=c.gbar, **c.kw), True)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step(g[:, 1:], w, m, v, hy, d=d, gbar_out=c.gbar, shard=shard, **c.kw), True)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step(g[::2], None, None, None, stats, **c.kw), True)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step(g, *(torch.nn.Parameter(t, requires_grad=False) for t in (w, m, v)), hy, d=7, gbar_out=c.gbar, **c.kw), True)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step_rows(rows, w, m, v, hy, table=table, gbar_out=c.gbar, **c.kw), True)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step_rows(tuple(rows), w, m, v, hy, table=table, d=d - 3, gbar_out=c.gbar, shard=shard, **c.kw), True)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step_clipped(g, w, m, v, c.gbar, 0.5, B.make_hyper(flags=FULL), d=d, **c.kw), True)
    c.same(monkeypatch, lambda w, m, v: B.normtest_adamw_gbar(rows[0].float(), w, m, v, hy, 0.25), True)
    c.same(monkeypatch, lambda w, m, v: B.normtest_adamw_gbar(rows[0].float(), w, m, v, hy, d=12), True)
    off = torch.tensor([0, 5, 1500, d], dtype=torch.int64, device="cuda")
    for lay in torch.zeros(3 * B.LAYER_BYTES, dtype=torch.uint8, device="cuda"), torch.zeros(400, dtype=torch.float64, device="cuda"):
        B.normtest_step(g, None, None, None, stats, d=d, **c.kw)
        tables, seen = [], _Recorded(B._fast)
        for fast in seen, None:
            with monkeypatch.context() as mp:
                mp.setattr(B, "_fast", fast)
                lay.zero_()
                assert B.normtest_layer_stats(g, off, c.ws, d=d, layers=lay) is lay
                tables.append(lay.clone())
        assert seen.back == [B.NT_OK]
        assert torch.equal(*(t.view(torch.int64) for t in tables)) and tables[0].any()
    # on another stream; what is left to Python: a stream of its own, numbers that are no plain int or float, subclasses of tensors
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        c.same(monkeypatch, lambda w, m, v: B.normtest_step(g, w, m, v, hy, d=d, gbar_out=c.gbar, **c.kw), True)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step(g, w, m, v, hy, d=d, gbar_out=c.gbar, stream=side, **c.kw), False)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step_clipped(g, w, m, v, c.gbar, 1, B.make_hyper(flags=FULL), d=d, **c.kw), False)
    c.same(monkeypatch, lambda w, m, v: B.normtest_adamw_gbar(rows[0].float(), w, m, v, hy, 1), False)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step(g.as_subclass(_Subclass), w, m, v, hy, d=d, gbar_out=c.gbar, **c.kw), False)
    c.same(monkeypatch, lambda w, m, v: B.normtest_step_rows(rows, w, m.as_subclass(_Subclass), v, hy, table=table, gbar_out=c.gbar, **c.kw), False)


class _Subclass(torch.Tensor):
    pass


# a graph of calls that the native call path has made, replayed between eager steps, and calls from several threads at once
@pytest.mark.gpu
def test_capture_and_threads(monkeypatch):
    B.lib()
    seen = _Recorded(B._fast)
    monkeypatch.setattr(B, "_fast", seen)
    hy = B.make_hyper(step=4, flags=FULL)
    c = _Gpu()
    state = [t.clone() for t in c.state]
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        B.normtest_step(c.grads, *state, hy, d=c.d, **c.kw)
    assert seen.back == [B.NT_OK]
    want = [t.clone() for t in c.state]
    res, ws = torch.zeros_like(c.res), torch.empty_like(c.ws)
    for _ in range(4):
        B.normtest_step(c.grads, *want, hy, d=c.d, workspace=ws, result=res)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((*state, c.res), (*want, res)))

    def steps(k, out):
        own = [t.clone() for t in c.state]
        r, w = torch.zeros_like(c.res), torch.empty_like(c.ws)
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.default_stream())
        with torch.cuda.stream(stream):
            back = [B._fast.fast.step(B.lib().normtest_step_entry, c.grads, *own, hy, c.d, None, None, w, r) for _ in range(40)]
        stream.synchronize()
        out[k] = (back == [B.NT_OK] * 40, own + [r])

    alone, outs = {}, {}
    steps(0, alone)
    threads = [threading.Thread(target=steps, args=(k, outs)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(outs) == 4 and alone[0][0] and all(ok for ok, _ in outs.values())
    assert all(torch.equal(a, b) for k in range(4) for a, b in zip(alone[0][1], outs[k][1]))


@pytest.mark.gpu
def test_what_is_refused_stays_refused(monkeypatch):
    c = _Gpu()
    g, d = c.grads, c.d
    hy = B.make_hyper(step=4, flags=FULL)
    rows = [r[:d].clone() for r in g]
    table = B.make_row_table(rows)
    bad = [lambda w, m, v: B.normtest_step(g, w.double(), m, v, hy, d=d, **c.kw), lambda w, m, v: B.normtest_step(g, w.cpu(), m, v, hy, d=d, **c.kw),
           lambda w, m, v: B.normtest_step(g, w, m, v, hy, **c.kw), lambda w, m, v: B.normtest_step(g.half(), w, m, v, hy, d=d, **c.kw),
           lambda w, m, v: B.normtest_step(g.t(), w, m, v, hy, d=5, **c.kw), lambda w, m, v: B.normtest_step(g[0], w, m, v, hy, d=d, **c.kw),
           lambda w, m, v: B.normtest_step(g, w, m, None, hy, d=d, **c.kw), lambda w, m, v: B.normtest_step(g, w, m[::2], v, hy, d=1000, **c.kw),
           lambda w, m, v: B.normtest_step(g, w, m, v, hy, d=-1, **c.kw), lambda w, m, v: B.normtest_step(g[:1], w, m, v, hy, d=d, **c.kw),
           lambda w, m, v: B.normtest_step(g, w, m, v, "hyper", d=d, **c.kw), lambda w, m, v: B.normtest_step(g, w, m, v, hy, d=2.5, **c.kw),
           lambda w, m, v: B.normtest_step(g, w, m, v, hy, d=d, workspace=c.ws[:64], result=c.res),
           lambda w, m, v: B.normtest_step(g, w, m, v, hy, d=d, workspace=c.ws[1:], result=c.res),
           lambda w, m, v: B.normtest_step_rows(rows[:2] + [rows[2][:9]], w, m, v, hy, d=d, table=table, **c.kw),
           lambda w, m, v: B.normtest_step_rows([rows[0], rows[1].float()], w, m, v, hy, table=table, **c.kw),
           lambda w, m, v: B.normtest_step_rows([g, g], w, m, v, hy, d=d, table=table, **c.kw),
           lambda w, m, v: B.normtest_step_clipped(g, w, m, v, None, 1.0, hy, d=d, **c.kw),
           lambda w, m, v: B.normtest_step_clipped(g, w, m, v, c.gbar, float("nan"), hy, d=d, **c.kw),
           lambda w, m, v: B.normtest_adamw_gbar(c.gbar, w, m, v, hy, float("inf")), lambda w, m, v: B.normtest_adamw_gbar(c.gbar, w, None, v, hy)]
    off = torch.tensor([0, 5, d], dtype=torch.int64, device="cuda")
    lay = torch.zeros(2 * B.LAYER_BYTES, dtype=torch.uint8, device="cuda")
    bad += [lambda w, m, v: B.normtest_layer_stats(g, off.int(), c.ws, d=d, layers=lay), lambda w, m, v: B.normtest_layer_stats(g, off[:1], c.ws, d=d, layers=lay),
            lambda w, m, v: B.normtest_layer_stats(g, off, c.ws[:200], d=d, layers=lay), lambda w, m, v: B.normtest_layer_stats(g, off, c.ws, d=d, layers=lay[:-1]),
            lambda w, m, v: B.normtest_layer_stats(g, off, c.ws.cpu(), d=d, layers=lay), lambda w, m, v: B.normtest_layer_stats(g, off[::2], c.ws, d=d, layers=lay),
            lambda w, m, v: B.normtest_layer_stats(g[:1], off, c.ws, d=d, layers=lay), lambda w, m, v: B.normtest_layer_stats(g.half(), off, c.ws, d=d, layers=lay)]
    for call in bad:
        c.same(monkeypatch, call, None, accepted=False)
