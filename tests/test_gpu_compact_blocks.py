"""Compaction with blocks of 32 rows (launches of up to two million rows) and of 64: rows copied bit for bit at the ends of
blocks and on either side of the rule."""
import numpy as np
import pytest
import torch

from paper_2605_06676_amd import lkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [[1], [31], [32], [33, 0, 31], [64, 1, 63, 65], [2 ** 20, 2 ** 20], [2 ** 20, 2 ** 20 + 1]])
def test_rows_arrive_whatever_the_block(lengths):
    ctx = lkv.Context(0)
    H, total = len(lengths), sum(lengths)
    T = max(lengths) + 3
    gen = torch.Generator(device="cuda").manual_seed(total)
    k, v = (torch.randint(-2 ** 15, 2 ** 15, (1, H, T, 128), dtype=torch.int16, device="cuda", generator=gen).view(torch.bfloat16)
            for _ in range(2))
    cache = lkv.Cache([k], [v], H)
    offsets = torch.empty(H + 1, dtype=torch.int32, device="cuda")
    assert lkv.lkv_plan_offsets(ctx, np.array(lengths, dtype=np.int32), offsets) == total
    idx = torch.cat([torch.randperm(T, device="cuda", generator=gen)[:m].sort().values for m in lengths]).int()
    kp, vp = (torch.zeros(total, 128, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    lkv.lkv_compact(ctx, cache, idx, offsets, total, kp, vp)
    at = 0
    for h, m in enumerate(lengths):
        rows = idx[at:at + m].long()
        for src, dst in ((k, kp), (v, vp)):
            assert torch.equal(src[0, h, rows].view(torch.int16), dst[at:at + m].view(torch.int16)), (h, m)
        at += m
    ctx.close()
