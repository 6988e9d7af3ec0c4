"""The sums over a tile's lanes and waves and over the tiles: small whole numbers, whose sums are exact in any order, so A, B, C
and the count of failing coordinates are compared for equality, at the edges of the batches in which tile partials are read."""
from __future__ import annotations

import pytest
import torch

from paper_2412_21124_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rows(J, d, gdtype, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randint(1, 5, (J, d), generator=g, device=DEV, dtype=torch.int8).to(gdtype)


def _sums(x):
    """A, B, C, failing coordinates and largest ratio for a threshold factor J - 1; every term is a multiple of 1/J"""
    J = x.shape[0]
    A = Bs = C = 0.0
    fail, worst = 0, 0.0
    for lo in range(0, x.shape[1], 1 << 22):
        y = x[:, lo:lo + (1 << 22)].double()
        s = y.sum(0)
        c = (y - s / J).square().sum(0)
        A, Bs, C = A + float(y.square().sum()), Bs + float(s.square().sum()), C + float(c.sum())
        den = (J - 1) * (s / J).square()
        fail += int((c > den).sum())
        worst = max(worst, float((c / den).max()))
    return A, Bs, C, fail, worst


def _hyper(J, flags):
    return B.make_hyper(lr=0.0, weight_decay=0.0, eta=1.0, step=1, b_k=1, round_to=1, ddof=1, flags=flags | B.NT_COORD_TEST)


# J, dtype, flags and the tile of that call; rows of 2 and 32 make every mean and every merge of two chunks exact
CALLS = [(2, torch.float32, B.NT_DO_STATS | B.NT_DO_ADAMW, 4096), (4, torch.bfloat16, B.NT_DO_STATS | B.NT_WRITE_GBAR, 4096),
         (32, torch.bfloat16, B.NT_DO_STATS, 2048)]


# one tile, less than a round of 256 partials, its edges, whole and part batches of eight rounds, both levels of reduction
@pytest.mark.parametrize("tiles", [1, 2, 63, 256, 257, 2047, 2048, 2049, 4096, 4097, 6145])
@pytest.mark.parametrize("J,gdtype,flags,tile", CALLS)
def test_sums_are_exact(J, gdtype, flags, tile, tiles):
    d = tiles * tile - (tiles % 3)
    x = _rows(J, d, gdtype, tiles)
    w, m, v, gbar = (torch.ones(d, device=DEV) for _ in range(4))
    res = B.read_result(B.normtest_step(x, w, m, v, _hyper(J, flags), gbar_out=gbar)).as_dict()
    A, Bs, C, fail, worst = _sums(x)
    assert (res["A"], res["B"], res["C"], res["coord_fail"]) == (A, Bs, C, fail)
    assert (res["A_lo"], res["B_lo"], res["C_lo"]) == (0.0, 0.0, 0.0)
    assert abs(res["coord_max_ratio"] - worst) <= 2.0 ** -22 * worst   # the kernel's fp32 product and quotient


# the per-layer table adds the same partials, whole groups of them through the group partials; layer ends inside tiles
def test_layer_sums_are_exact():
    J, tile = 2, 4096
    d = 6145 * tile + 77
    x = _rows(J, d, torch.float32, 5)
    w, m, v = (torch.ones(d, device=DEV) for _ in range(3))
    edges = [0, 1, 5 * tile, 5 * tile + 3, 1030 * tile - 1, 4097 * tile + 9, d]
    ws = torch.empty(B.normtest_workspace_bytes(J, d), dtype=torch.uint8, device=DEV)
    B.normtest_step(x, w, m, v, _hyper(J, B.NT_DO_STATS | B.NT_DO_ADAMW), workspace=ws)
    table = B.normtest_layer_stats(x, torch.tensor(edges, dtype=torch.int64, device=DEV), ws)
    for got, lo, hi in zip(B.read_layers(table), edges[:-1], edges[1:]):
        A, Bs, C, fail, _ = _sums(x[:, lo:hi])
        assert (got.A, got.B, got.C, got.coord_fail) == (A, Bs, C, fail)


# one block for all tiles and a block per group of them; groups of 512 tiles, the last one whole, short or a single tile, and of 2048
@pytest.mark.parametrize("tiles", [2559, 2560, 2561, 3072, 3073, 9000, (1 << 16) - 1, 1 << 16, (1 << 16) + 1])
def test_sums_are_exact_over_groups_of_tiles(tiles):
    d = tiles * 4096 - (tiles % 3)
    x = _rows(2, d, torch.bfloat16, tiles)
    gbar = torch.empty(d, device=DEV)
    ws = torch.randint(0, 255, (B.normtest_workspace_bytes(2, d),), dtype=torch.uint8, device=DEV)
    A, Bs, C, fail, _ = _sums(x)
    for _ in range(3):   # the counter in the workspace is as the call before left it
        res = B.read_result(B.normtest_step(x, None, None, None, _hyper(2, B.NT_DO_STATS | B.NT_WRITE_GBAR), gbar_out=gbar, workspace=ws))
        assert (res.A, res.B, res.C, res.coord_fail) == (A, Bs, C, fail)
    cut = [0, 5, 512 * 4096, 512 * 4096 + 1, 2048 * 4096, 2400 * 4096 - 7, d]
    layers = B.read_layers(B.normtest_layer_stats(x, torch.tensor(cut, dtype=torch.int64, device=DEV), ws))
    for got, lo, hi in zip(layers, cut[:-1], cut[1:]):
        want = _sums(x[:, lo:hi])
        assert (got.A, got.B, got.C, got.coord_fail) == want[:4], (lo, hi)


# a workspace whose record names another number of groups, as one kept from a build with groups of 2048 tiles: the table reads its tiles
def test_groups_of_another_size_are_not_read():
    d = 9000 * 4096
    x = _rows(2, d, torch.bfloat16, 3)
    gbar = torch.empty(d, device=DEV)
    ws = torch.zeros(B.normtest_workspace_bytes(2, d), dtype=torch.uint8, device=DEV)
    off = torch.tensor([0, 7 * 2048, 2048 * 4096, 8999 * 4096 + 5, d], dtype=torch.int64, device=DEV)
    B.normtest_step(x, None, None, None, _hyper(2, B.NT_DO_STATS | B.NT_WRITE_GBAR), gbar_out=gbar, workspace=ws)
    want = B.normtest_layer_stats(x, off, ws).clone()
    record = ws.view(torch.int64)
    ntiles = int(record[2])
    assert int(record[3]) == -(-ntiles // 512)
    record[3] = -(-ntiles // 2048)
    ws.view(torch.float64)[32 + 5 * ntiles:] = float("nan")
    assert torch.equal(B.normtest_layer_stats(x, off, ws), want)


# the counter is in the workspace, so a graph takes the same kernels; replayed with other inputs and eager steps of other sizes between
def test_groups_of_tiles_in_a_graph():
    d = 2600 * 4096 - 1
    x = _rows(2, d, torch.float32, 1)
    state = [torch.ones(d, device=DEV) for _ in range(3)]
    ws = torch.randint(0, 255, (B.normtest_workspace_bytes(2, d),), dtype=torch.uint8, device=DEV)
    res = torch.zeros(B.RESULT_BYTES, dtype=torch.uint8, device=DEV)
    hy = _hyper(2, B.NT_DO_STATS | B.NT_DO_ADAMW)

    def step():
        return B.normtest_step(x, *state, hy, workspace=ws, result=res)

    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        step()
    for k in range(4):
        x.copy_(_rows(2, d, torch.float32, 10 + k))
        graph.replay()
        torch.cuda.synchronize()
        got = res.clone()
        res.zero_()
        B.normtest_step(x, *state, hy, d=4096 * (k + 1), workspace=ws, result=res)
        step()
        torch.cuda.synchronize()
        assert torch.equal(got, res)
        A, Bs, C, fail, _ = _sums(x)
        r = B.read_result(got)
        assert (r.A, r.B, r.C, r.coord_fail) == (A, Bs, C, fail)
