"""Shared block and suffix in one launch (combined_impl.h): the calls that take it (a level with more than 128 query rows
on the persistent kernel; the planner's view says which cells those are) over every suffix cache, at the edges of its batches, chunks, pages and runs of
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
    "four_levels": (300, 1, 128, [(1, 40, 300), (2, 65, 150), (3, 33, 100), (1, 64, 280)], 0, 20),
    "several_blocks": (600, 2, 64, [(3, 90, 200)], 0, 50),
    "many_items": (1300, 10, 128, [(1, 40, 1300)], 1, 24),
    "many_sequences": (15400, 1, 64, [(1, 33, 15400)], 0, 6),        # more sequences than the table of their order holds
}


# several query rows per KV head; name: (B, query heads, KV heads, D, queries per sequence, levels, suffix lengths)
TILE_SHAPES = {
    "g8": (40, 16, 2, 128, 1, [(1, 97, 40)], 0, 70),
    "g16": (33, 16, 1, 128, 1, [(1, 64, 33)], 31, 65),              # a full 16-row tile
    "g3_nq6": (24, 6, 2, 128, 6, [(1, 40, 24)], 0, 45),             # 18 rows: a 32-row tile, causal among the new tokens
    "two_tiles": (9, 40, 1, 128, 1, [(1, 70, 9)], 1, 40),           # 40 rows: two 32-row tiles, the second partly filled
    "nq2": (150, 3, 3, 128, 2, [(1, 130, 150)], 0, 34),
    "g8_d64": (40, 16, 2, 64, 1, [(1, 97, 40)], 0, 70),
    "nq5_d64": (60, 8, 2, 64, 5, [(1, 97, 60)], 0, 50),
    "one_row": (400, 1, 1, 128, 1, [(1, 70, 400)], 0, 390),         # long suffixes with one row per KV head
    "tile_chunks": (70, 8, 2, 128, 1, [(2, 60, 35)], 0, 1100),
    "tile_levels": (200, 8, 2, 128, 1, [(1, 200, 200), (8, 33, 25)], 0, 20),
    "tile_items": (1100, 8, 4, 128, 1, [(1, 40, 1100)], 1, 24),     # two rows per KV head and short suffixes: separate kernels
    "tile_items_g4": (1100, 16, 4, 128, 1, [(1, 40, 1100)], 1, 24),
}


def takes_combined_launch(shape, cache, slots):
    """What the automatic choice makes of a cell: 8-bit rows in 32-row tiles or on the vector ALU with several rows per KV head
    keep separate kernels, and so do short suffixes of one row per KV head unless the CUs of the shared block are set."""
    codes = cache in ("fp8", "paged_fp8", "paged_fp8_16")
    if shape in SHAPES:
        return slots > 0 or SHAPES[shape][5] >= (24 if not codes else 48 if SHAPES[shape][3] == 128 else 80)
    B, H, Hkv, D, nq = TILE_SHAPES[shape][:5]
    if shape == "tile_items":
        return False
    return not codes or (D == 128 and nq * H // Hkv <= 16)


@pytest.mark.parametrize("cache", ["packed", "paged", "fp8", "paged_fp8", "paged_fp8_16"])
@pytest.mark.parametrize("shape", [*SHAPES, *TILE_SHAPES])
def test_combined(shape, cache):
    if shape in SHAPES:
        B, H, D, levels, lo, hi = SHAPES[shape]
        Hkv, nq = H, 1
    else:
        B, H, Hkv, D, nq, levels, lo, hi = TILE_SHAPES[shape]
    print(f"combined: {shape} {cache} B={B} {H}/{Hkv} D={D} nq={nq} {levels} {lo}..{hi}", file=sys.stderr, flush=True)
    w = wl.make_workload(shape, 77, B, H, Hkv, D, levels, lo, hi, nq=nq)
    w.lengths[:2] = (hi, lo)           # the longest and the shortest are there
    w = wl.make_workload(shape, 77, B, H, Hkv, D, levels, lo, hi, lengths=np.ascontiguousarray(w.lengths), nq=nq)
    dw = dev.to_device(w)
    Oref, Lref, call = reference(w, cache)
    ctx = dev.make_context(dw, parts=32)
    ctx.set_option(hb.HG_OPT_FUSED_KERNEL, 1)       # (not the single launch of small calls)
    for slots in (0, 4, 32):                        # workgroups per XCD that take the shared block first
        ctx.set_option(hb.HG_OPT_WIDE_SLOTS, slots)
        page = {"paged": 16, "paged_fp8": 32, "paged_fp8_16": 16}.get(cache, 0)
        plan = hb.hg_debug_fused_plan(levels, B, nq, H, Hkv, D, dw.max_len, page, "fp8" in cache,
                                      hb.hg_workspace_bytes(B * nq, H, D, 32), {hb.HG_OPT_FUSED_KERNEL: 1, hb.HG_OPT_WIDE_SLOTS: slots})
        assert (plan["way"] == "combined") == takes_combined_launch(shape, cache, slots), plan
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


@pytest.mark.parametrize("cache", ["packed", "paged", "fp8", "paged_fp8"])
@pytest.mark.parametrize("B,H,D", [(200, 480, 128), (2400, 40, 128), (15000, 7, 128), (200, 880, 64), (4200, 40, 64), (15360, 9, 64)])
def test_combined_more_results_than_a_wavefront_keeps(B, H, D, cache):
    """More work items per wavefront than results fit its LDS: in the 16 KiB of the ring's memory, then behind the order of the sequences (7, 6 and
    no rows at D = 128, 14, 10 and none at D = 64), then each written at once."""
    row = 4 * D + 16
    kept = 16384 // row + max(0, 32768 - 512 - 2 * B) // (8 * row)
    assert B * H > 1.1 * 2048 * kept
    print(f"combined, results: {cache} B={B} H={H} D={D} {kept} kept", file=sys.stderr, flush=True)
    w = wl.make_workload("kept", 79, B, H, H, D, [(1, 33, B)], 1, 3)
    dw = dev.to_device(w)
    Oref, Lref, call = reference(w, cache)
    ctx = dev.make_context(dw, parts=8)
    ctx.set_option(hb.HG_OPT_WIDE_SLOTS, 4)
    plan = hb.hg_debug_fused_plan([(1, 33, B)], B, 1, H, H, D, dw.max_len, {"paged": 16, "paged_fp8": 32}.get(cache, 0), "fp8" in cache,
                                  hb.hg_workspace_bytes(B, H, D, 8), {hb.HG_OPT_FUSED_KERNEL: 1, hb.HG_OPT_WIDE_SLOTS: 4})
    assert plan["way"] == "combined" and plan["nchunks"] == 1, plan
    got = []
    for _ in range(2):
        O = torch.full(dw.lead + (dw.D,), float("nan"), dtype=torch.float32, device="cuda:0")
        L = torch.full(dw.lead, float("nan"), dtype=torch.float32, device="cuda:0")
        call(ctx, dw, O, L)
        got.append((O, L))
    torch.cuda.synchronize()
    check(to_np(got[0][0]), to_np(got[0][1]), Oref, Lref, f"kept results {cache} B={B} H={H} D={D}")
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    ctx.close()


@pytest.mark.parametrize("cache", ["packed", "paged"])
@pytest.mark.parametrize("heads", [1, 8])
@pytest.mark.parametrize("B", [129, 223, 224, 225, 448, 1000, 1791, 1792, 1793, 2048, 2817])
def test_combined_item_runs(B, heads, cache):
    """One work item per sequence, on the vector ALU and the matrix cores: fewer than the 224 (256) workgroups that start with a run, as many, one more, runs of
    2 to 8, first runs that leave no items, one, and a tail behind long runs."""
    print(f"combined, runs: {cache} B={B} heads={heads}", file=sys.stderr, flush=True)
    w = wl.make_workload("runs", 80, B, heads, 1, 128, [(1, 40, B)], 0, 40)
    dw = dev.to_device(w)
    Oref, Lref, call = reference(w, cache)
    ctx = dev.make_context(dw, parts=16)
    ctx.set_option(hb.HG_OPT_FUSED_KERNEL, 1)
    for slots in (4, 32):
        ctx.set_option(hb.HG_OPT_WIDE_SLOTS, slots)
        plan = hb.hg_debug_fused_plan([(1, 40, B)], B, 1, heads, 1, 128, dw.max_len, 16 if cache == "paged" else 0, False, hb.hg_workspace_bytes(B, heads, 128, 16),
                                      {hb.HG_OPT_FUSED_KERNEL: 1, hb.HG_OPT_WIDE_SLOTS: slots})
        assert (plan["way"], plan["nchunks"], plan["mfma"]) == ("combined", 1, int(heads > 1)), plan
        got = []
        for _ in range(2):
            O = torch.full(dw.lead + (128,), float("nan"), dtype=torch.float32, device="cuda:0")
            L = torch.full(dw.lead, float("nan"), dtype=torch.float32, device="cuda:0")
            call(ctx, dw, O, L)
            got.append((O, L))
        torch.cuda.synchronize()
        check(to_np(got[0][0]), to_np(got[0][1]), Oref, Lref, f"runs {cache} B={B} heads={heads} slots={slots}")
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    ctx.close()


@pytest.mark.parametrize("shape", ["many_items", "tile_items", "tile_items_g4"])
def test_combined_capture(shape):
    """Captured once, replayed with eager calls and other inputs in between: every replay leaves its counters at zero."""
    if shape in SHAPES:
        B, H, D, levels, lo, hi = SHAPES[shape]
        Hkv, nq = H, 1
    else:
        B, H, Hkv, D, nq, levels, lo, hi = TILE_SHAPES[shape]
    print(f"combined, captured: {shape}", file=sys.stderr, flush=True)
    dw = dev.to_device(wl.make_workload(shape, 78, B, H, Hkv, D, levels, lo, hi, nq=nq))
    ctx = dev.make_context(dw, parts=32)
    ctx.set_option(hb.HG_OPT_FUSED_KERNEL, 1)
    ctx.set_option(hb.HG_OPT_WIDE_SLOTS, 12)
    way = hb.hg_debug_fused_plan(levels, B, nq, H, Hkv, D, dw.max_len, options={hb.HG_OPT_FUSED_KERNEL: 1, hb.HG_OPT_WIDE_SLOTS: 12})["way"]
    assert (way == "combined") == takes_combined_launch(shape, "packed", 12)
    O = torch.empty(dw.lead + (dw.D,), dtype=torch.float32, device="cuda:0")
    L = torch.empty(dw.lead, dtype=torch.float32, device="cuda:0")

    def call(o, l):
        hb.hg_hydragen_attn(ctx, dw.Q, dw.levels, dw.Ks, dw.Vs, dw.offsets, dw.lengths, dw.max_len, o, l, dw.scale)

    call(O, L)
    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ctx.set_stream(side)
        call(O, L)
    ctx.set_stream(None)
    for _ in range(3):
        dw.Q.copy_(torch.randn_like(dw.Q))
        Oe, Le = torch.empty_like(O), torch.empty_like(L)
        call(Oe, Le)
        torch.cuda.synchronize()
        O.fill_(float("nan"))
        L.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(O, Oe) and torch.equal(L, Le), f"{shape}: a replay differs from the eager call"
    ctx.close()
