"""More than 16 bf16 rows in a matrix of odd row stride, whose every second row is loaded in words and shifted, against the same rows
with an even stride: every output has to have the same bits, where a sweep ends before, at and behind the last coordinate."""
from __future__ import annotations

import pytest
import torch

from paper_2412_21124_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STATS, ADAMW, GBAR, COORD = B.NT_DO_STATS, B.NT_DO_ADAMW, B.NT_WRITE_GBAR, B.NT_COORD_TEST


# the classes of tiles by the length of the whole vector; the first matrix row on a word (shift 0) and between two
@pytest.mark.parametrize("whole", [1 << 18, 1 << 19, 1 << 22, 1 << 26])
@pytest.mark.parametrize("J,flags", [(17, STATS | ADAMW | COORD), (32, STATS), (33, ADAMW), (48, STATS | ADAMW), (64, STATS | GBAR), (131, STATS | ADAMW), (128, ADAMW | GBAR)])
def test_bits_of_an_even_stride(J, flags, whole):
    g = torch.Generator(device=DEV).manual_seed(J)
    hy = B.make_hyper(lr=3e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1, step=5, b_k=64, b_max=8192, round_to=8, flags=flags)
    shard = B.nt_shard_info(0, 8, 0, whole)
    for d, gap in [(1, 0), (255, 0), (257, 0), (1025, 0), (2047, 0), (2048, 1), (2049, 0), (8191, 2), (8192, 1), (8193, 0), (16385, 6), (20481, 0)]:
        ld = d + gap
        for shift in (0, 1):
            flat = (torch.randn(J * ld + shift, generator=g, device=DEV) * 1e-2).to(torch.bfloat16)
            odd = flat[shift:].view(J, ld)
            even = torch.empty(J, (ld + 63) // 64 * 64, dtype=torch.bfloat16, device=DEV)
            even[:, :d] = odd[:, :d]
            state = [torch.rand(d, generator=g, device=DEV) * 0.02 for _ in range(4)]
            outs = []
            for rows in (odd, even):
                st = [s.clone() for s in state]
                res = B.normtest_step(rows, *st[:3], hy, d=d, gbar_out=st[3] if flags & GBAR else None, shard=shard)
                outs.append([B.read_result(res).as_dict()] + st)
            for x, y in zip(outs[0][1:], outs[1][1:]):
                assert torch.equal(x, y), (d, shift)
            if flags & STATS:
                for k in ("A", "B", "C", "T", "coord_fail", "coord_max_ratio"):
                    assert outs[0][0][k] == outs[1][0][k], (d, shift, k)
