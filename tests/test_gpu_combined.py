"""Shared block and suffix in one launch (combined_impl.h): the calls that take it (a level with more than 128 query rows
on the persistent kernel) over every suffix cache, at the edges of its batches, chunks, pages and runs of
work items, against the fp64 oracle.  Every call runs twice in a row: the first must leave its work counter at zero."""
import sys

import numpy as np
import pytest
import torch

from paper_2402_05099_amd import binding as hb
from paper_2402_05099_amd import device as dev
from paper_2402_05099_amd import workloads as wl
from parity import check, to_np
from test_gpu_split_launch import reference

pytestmark = pytest.mark.gpu

# name: (B, heads, D, levels, suffix lengths (lo, hi))
SHAPES = {
    "one_row_over": (129, 1, 128, [(1, 31, 129)], 1, 1),
    "batch_edges": (300, 3, 128, [(1, 100, 300)], 14, 34),
    "batch_edges_d64": (300, 3, 64, [(1, 100, 300)], 30, 66),
    "chunks": (140, 2, 128, [(1, 257, 140)], 0, 383),
    "chunks_d64": (140, 2, 64, [(1, 257, 140)], 0, 700),
    "two_levels": (320, 2, 128, [(1, 200, 320), (4, 65, 80)], 0, 20),
    "several_blocks": (600, 2, 64, [(3, 90, 200)], 0, 50),
    "many_items": (1300, 10, 128, [(1, 40, 1300)], 1, 24),
}


@pytest.mark.parametrize("cache", ["packed", "paged", "fp8", "paged_fp8"])
@pytest.mark.parametrize("shape", SHAPES)
def test_combined(shape, cache):
    B, H, D, levels, lo, hi = SHAPES[shape]
    print(f"combined: {shape} {cache} {SHAPES[shape]}", file=sys.stderr, flush=True)
    w = wl.make_workload(shape, 77, B, H, H, D, levels, lo, hi)
    w.lengths[:2] = (hi, lo)           # the longest and the shortest are there
    w = wl.make_workload(shape, 77, B, H, H, D, levels, lo, hi, lengths=np.ascontiguousarray(w.lengths))
    dw = dev.to_device(w)
    Oref, Lref, call = reference(w, cache)
    ctx = dev.make_context(dw, parts=32)
    ctx.set_option(hb.HG_OPT_FUSED_KERNEL, 1)       # (not the single launch of small calls)
    for slots in (0, 4, 32):                        # workgroups per XCD that take the shared block first
        ctx.set_option(hb.HG_OPT_WIDE_SLOTS, slots)
        got = []
        for _ in range(2):
            O = torch.full(dw.lead + (dw.D,), float("nan"), dtype=torch.float32, device="cuda:0")
            L = torch.full(dw.lead, float("nan"), dtype=torch.float32, device="cuda:0")
            call(ctx, dw, O, L)
            got.append((O, L))
        torch.cuda.synchronize()
        check(to_np(got[0][0]), to_np(got[0][1]), Oref, Lref, f"{shape} {cache} slots={slots}")
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), f"{shape} {cache}: the second call differs"
    ctx.close()
