"""Steps of a few tiles, whose last block adds up the partials: the bits of the two launches that the same call takes under
capture, with inputs that change from call to call, garbage in the workspace, and several streams at once."""
from __future__ import annotations

import ctypes
import threading

import pytest
import torch

import helpers as H
from paper_2412_21124_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STATS, ADAMW, GBAR, COORD = B.NT_DO_STATS, B.NT_DO_ADAMW, B.NT_WRITE_GBAR, B.NT_COORD_TEST
K = 4   # inputs, and streams


def _hyper(flags, **kw):
    # without lr, decay and betas every call on the same inputs leaves the same state: w as it is, m = g, v = g^2
    kw = {"lr": 0.0, "weight_decay": 0.0, "beta1": 0.0, "beta2": 0.0, **kw}
    return B.make_hyper(step=10, b_k=64, b_max=8192, round_to=16, flags=flags, **kw)


class _Calls:
    """K inputs of one size, each with a state, a workspace full of garbage and a pointer table of its own."""
    def __init__(self, J, gdtype, d, flags, whole=0):
        self.hy, self.d = _hyper(flags), d
        self.shard = B.nt_shard_info(0, 1, 0, whole) if whole else None   # a part of a longer vector
        self.grads = [(torch.randn(J, d, device=DEV) * 1e-2 * (k + 1)).to(gdtype) for k in range(K)]
        self.rows = [[g[j] for j in range(J)] for g in self.grads]
        self.tables = [B.make_row_table(r) for r in self.rows]
        self.state = [[torch.rand(d, device=DEV) for _ in range(4)] for _ in range(K)]
        self.ws = [torch.randint(0, 255, (B.normtest_workspace_bytes(J, d),), dtype=torch.uint8, device=DEV) for _ in range(K)]

    def matrix(self, k, result, stream=None):
        w, m, v, gbar = self.state[k]
        B.normtest_step(self.grads[k], w, m, v, self.hy, shard=self.shard, gbar_out=gbar, workspace=self.ws[k], result=result,
                        stream=stream)

    def table(self, k, result, stream=None):
        w, m, v, gbar = self.state[k]
        B.normtest_step_rows(self.rows[k], w, m, v, self.hy, table=self.tables[k], shard=self.shard, gbar_out=gbar,
                             workspace=self.ws[k], result=result, stream=stream)

    def reset(self):
        """Values that no call leaves behind, so that a store left out shows."""
        for w, *rest in self.state:
            w.copy_(torch.linspace(0.5, 1.5, self.d, device=DEV))
            for t in rest:
                t.fill_(7.0)
        torch.cuda.synchronize()

    def two_launches(self):
        """Result and outputs for every input from a captured step, which has a reduction kernel of its own."""
        self.reset()
        out = []
        for k in range(K):
            r = torch.zeros(B.RESULT_BYTES, dtype=torch.uint8, device=DEV)
            H.captured(lambda: self.matrix(k, r))
            out.append((r, [t.clone() for t in self.state[k]]))
        return out

    def check(self, want):
        torch.cuda.synchronize()
        for k in range(K):
            assert all(torch.equal(a, b) for a, b in zip(self.state[k], want[k][1])), k


# the fewest tiles, a ragged last one, both sides of the last count that ends in one launch, for each class of short vectors and,
# beyond 16 rows, of short tiles
@pytest.mark.parametrize("J,gdtype,flags,tile,most,whole", [
    (2, torch.float32, STATS | ADAMW, 4096, 256, 0), (16, torch.bfloat16, STATS, 4096, 512, 0),
    (8, torch.bfloat16, STATS | GBAR | COORD, 4096, 512, 0), (20, torch.float32, STATS | ADAMW | GBAR, 2048, 128, 0),
    (40, torch.bfloat16, STATS, 2048, 128, 0), (24, torch.bfloat16, STATS | ADAMW | GBAR, 2048, 128, 1 << 22),
    (33, torch.float32, STATS | GBAR, 2048, 128, 1 << 22), (19, torch.float32, STATS, 2048, 128, 1 << 30)])
@pytest.mark.parametrize("past", [None, -1, 0, 1])
def test_bits_of_two_launches(J, gdtype, flags, tile, most, whole, past):
    tiles = 2 if past is None else most + past
    c = _Calls(J, gdtype, tiles * tile - 5, flags, whole)
    want = c.two_launches()
    c.reset()
    results = torch.zeros(2 * K * 20, B.RESULT_BYTES, dtype=torch.uint8, device=DEV)
    for i in range(results.shape[0]):   # back to back, every input after another one
        (c.matrix if i % (2 * K) < K else c.table)(i % K, results[i])
    c.check(want)
    assert all(torch.equal(results[i], want[i % K][0]) for i in range(results.shape[0]))
    c.reset()
    results.zero_()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(K)]
    for i in range(results.shape[0]):
        c.matrix(i % K, results[i], streams[i % K])
    c.check(want)
    assert all(torch.equal(results[i], want[i % K][0]) for i in range(results.shape[0]))
    # one step that moves every part of the state
    c.hy = _hyper(flags, lr=3e-2, weight_decay=0.1, beta1=0.9, beta2=0.95)
    want = c.two_launches()
    for way in (c.matrix, c.table):
        c.reset()
        for k in range(K):
            way(k, results[k])
        c.check(want)


# both sides of the count from which the blocks count themselves in several counters, one more than a round of those, and of the
# last counts that end in one launch
@pytest.mark.parametrize("J,gdtype,flags,tile,tiles", [
    (3, torch.bfloat16, STATS | ADAMW, 4096, (96, 97, 104, 105, 256)), (6, torch.float32, STATS | GBAR | COORD, 4096, (97, 511, 512, 513)),
    (9, torch.bfloat16, STATS, 4096, (103, 511)), (23, torch.float32, STATS | ADAMW, 1024, (96, 97, 255, 256, 257)),
    (50, torch.bfloat16, STATS | GBAR, 1024, (97, 256, 257))])
def test_bits_of_two_launches_with_several_counters(J, gdtype, flags, tile, tiles):
    for n in tiles:
        c = _Calls(J, gdtype, n * tile - 5, flags)
        want = c.two_launches()
        c.reset()
        results = torch.zeros(6 * K, B.RESULT_BYTES, dtype=torch.uint8, device=DEV)
        for i in range(results.shape[0]):
            c.matrix(i % K, results[i])
        c.check(want)
        assert all(torch.equal(results[i], want[i % K][0]) for i in range(results.shape[0])), n


# Sums that are not finite: the last block's totals against the reduction kernel's, an infinite row and squares that overflow
@pytest.mark.parametrize("J,gdtype,tile", [(2, torch.float32, 4096), (16, torch.bfloat16, 4096), (33, torch.float32, 2048)])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 1e20])
def test_sums_that_are_not_finite(J, gdtype, tile, value):
    for tiles in (2, 100):
        c = _Calls(J, gdtype, tiles * tile - 3, STATS | ADAMW | GBAR | COORD)
        for g in c.grads:
            g[:1 if value != 1e20 else J, tile + 7] = value
        want = c.two_launches()
        got = torch.zeros(2 * K, B.RESULT_BYTES, dtype=torch.uint8, device=DEV)
        c.reset()
        for k in range(K):
            c.matrix(k, got[k])
        for k in range(K):
            c.table(k, got[K + k])
        torch.cuda.synchronize()
        assert B.read_result(got[0]).status == B.NT_STATUS_NONFINITE
        # every word of the record, NaN by its bits
        assert all(torch.equal(got[k], want[k % K][0]) for k in range(2 * K))


# the default stream that every thread has of its own goes by one handle (2) in all of them
def test_threads_own_streams():
    c = _Calls(4, torch.float32, 200 * 4096 - 5, STATS | ADAMW | GBAR)
    want = c.two_launches()
    c.reset()
    results = torch.zeros(K, 50, B.RESULT_BYTES, dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    fn, codes = B.lib().normtest_step, {}

    def calls(k):
        w, m, v, gbar = (t.data_ptr() for t in c.state[k])
        codes[k] = [fn(c.grads[k].data_ptr(), B.NT_F32, 4, c.d, c.d, w, m, v, gbar, ctypes.byref(c.hy), None, c.ws[k].data_ptr(),
                       c.ws[k].numel(), results[k, i].data_ptr(), 2) for i in range(50)]
        torch.cuda.synchronize()

    threads = [threading.Thread(target=calls, args=(k,)) for k in range(K)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert codes == {k: [0] * 50 for k in range(K)}
    c.check(want)
    assert all(torch.equal(results[k, i], want[k][0]) for k in range(K) for i in range(50))


# more calls than the counters of all streams: the stream's own is met by each and left at zero
def test_counters_come_round():
    c = _Calls(2, torch.float32, 4097, STATS)
    want = c.two_launches()[0][0]
    res = torch.zeros(B.RESULT_BYTES, dtype=torch.uint8, device=DEV)
    fn = B.lib().normtest_step
    args = (c.grads[0].data_ptr(), B.NT_F32, 2, c.d, c.d, None, None, None, None, ctypes.byref(c.hy), None, c.ws[0].data_ptr(),
            c.ws[0].numel(), res.data_ptr(), torch.cuda.current_stream().cuda_stream)
    for i in range((1 << 20) + 5):
        if fn(*args) != 0:
            raise AssertionError(i)
        if i % (1 << 17) == 0:
            print("call", i, flush=True)
            torch.cuda.synchronize()
            assert torch.equal(res, want)
            res.zero_()
    torch.cuda.synchronize()
    assert torch.equal(res, want)
