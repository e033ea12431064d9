"""The single launch with columns of 16 and of 32 query rows, asked for by option, over every suffix cache: rows around the ends
of a column, numbers of KV heads that divide the XCDs evenly and that do not, block boundaries inside a column, runs of
stages that end in the shared rows and in the suffixes.  Against the fp64 oracle; without a workspace and with one (columns
of paged and 8-bit calls are then split over workgroups); twice in a row with the same bits."""
import sys

import pytest
import torch

from paper_2402_05099_amd import binding as hb
from paper_2402_05099_amd import device as dev
from paper_2402_05099_amd import workloads as wl
from parity import check, to_np
from test_gpu_split_launch import reference

pytestmark = pytest.mark.gpu

# name: (B, query heads, KV heads, D, queries per sequence, levels (blocks, rows, sequences per block), suffix lengths)
SHAPES = {
    "one_row": (1, 1, 1, 128, 1, [(1, 1, 1)], 1, 1),
    "rows_15": (15, 3, 3, 128, 1, [(1, 33, 15)], 1, 40),             # three KV heads: eighths that end inside a head
    "rows_17": (17, 2, 2, 64, 1, [(1, 300, 17)], 0, 33),
    "rows_33": (11, 24, 8, 128, 1, [(1, 31, 11)], 1, 65),            # a sequence's rows cross the end of a column; one KV head per XCD
    "group_of_5": (7, 10, 2, 128, 1, [(1, 97, 7)], 0, 90),
    "group_of_32": (3, 64, 2, 128, 1, [(1, 40, 3)], 5, 64),
    "queries": (9, 8, 8, 64, 5, [(1, 64, 9)], 2, 70),                # causal among the new tokens
    "block_edges": (50, 4, 4, 128, 1, [(1, 20, 50), (7, 35, 7)], 0, 20),      # boundaries inside columns, a sequence no block covers
    "no_shared": (40, 16, 16, 128, 1, [], 0, 50),                    # two KV heads per XCD
    "shared_only_first": (20, 4, 1, 128, 1, [(1, 700, 20)], 0, 1),   # more shared stages than wavefronts, hardly a suffix
}


@pytest.mark.parametrize("cache", ["packed", "paged", "fp8", "paged_fp8_16"])
@pytest.mark.parametrize("rows", [16, 32])
@pytest.mark.parametrize("shape", SHAPES)
def test_columns(shape, rows, cache):
    B, H, Hkv, D, nq, levels, lo, hi = SHAPES[shape]
    print(f"columns: {shape} rows={rows} {cache}", file=sys.stderr, flush=True)
    w = wl.make_workload(shape, 91, B, H, Hkv, D, levels, lo, hi, nq=nq)
    dw = dev.to_device(w)
    Oref, Lref, call = reference(w, cache)
    for parts in (32, 0):
        ctx = dev.make_context(dw, parts=parts) if parts else hb.Context(0, 0)
        ctx.set_option(hb.HG_OPT_FUSED_KERNEL, 2)
        ctx.set_option(hb.HG_OPT_SUFFIX_TILE_ROWS, rows)
        got = []
        for _ in range(2):
            O = torch.full(dw.lead + (dw.D,), float("nan"), dtype=torch.float32, device="cuda:0")
            L = torch.full(dw.lead, float("nan"), dtype=torch.float32, device="cuda:0")
            call(ctx, dw, O, L)
            got.append((O, L))
        torch.cuda.synchronize()
        check(to_np(got[0][0]), to_np(got[0][1]), Oref, Lref, f"{shape} rows={rows} {cache} parts={parts}")
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
        ctx.close()


# suffixes that keep the HBM busy while the chip holds one round of columns: a wavefront's stages are then consecutive
RUN_SHAPES = {
    "runs": (820, 8, 1, 128, 1, [(1, 70, 820)], 0, 260),
    "runs_blocks": (500, 16, 2, 128, 1, [(1, 40, 500), (7, 35, 71)], 0, 300),      # boundaries inside columns, sequences no block covers
    "runs_queries": (210, 8, 1, 128, 4, [(1, 64, 210)], 4, 700),
    "runs_no_shared": (800, 8, 1, 128, 1, [], 1, 300),
}


@pytest.mark.parametrize("cache", ["packed", "paged"])
@pytest.mark.parametrize("shape", RUN_SHAPES)
def test_stages_in_runs(shape, cache):
    B, H, Hkv, D, nq, levels, lo, hi = RUN_SHAPES[shape]
    print(f"stages in runs: {shape} {cache}", file=sys.stderr, flush=True)
    w = wl.make_workload(shape, 92, B, H, Hkv, D, levels, lo, hi, nq=nq)
    dw = dev.to_device(w)
    Oref, Lref, call = reference(w, cache)
    options = {hb.HG_OPT_FUSED_KERNEL: 2, hb.HG_OPT_SUFFIX_TILE_ROWS: 32}
    plan = hb.hg_debug_fused_plan(levels, B, nq, H, Hkv, D, dw.max_len, 16 if cache == "paged" else 0, options=options)
    assert (plan["way"], plan["dealt"]) == ("single", False)
    ctx = dev.make_context(dw, parts=32)
    for option, value in options.items():
        ctx.set_option(option, value)
    got = []
    for _ in range(2):
        O = torch.full(dw.lead + (dw.D,), float("nan"), dtype=torch.float32, device="cuda:0")
        L = torch.full(dw.lead, float("nan"), dtype=torch.float32, device="cuda:0")
        call(ctx, dw, O, L)
        got.append((O, L))
    torch.cuda.synchronize()
    check(to_np(got[0][0]), to_np(got[0][1]), Oref, Lref, f"{shape} {cache}")
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    ctx.close()


# more columns than CUs, few stages to a column: workgroups of four wavefronts
FOUR_SHAPES = {
    "one_tile_more": (1028, 8, 8, 128, 1, [(1, 33, 1028)], 1, 40),
    "block_edges": (700, 12, 12, 128, 1, [(1, 20, 700), (7, 35, 100)], 0, 20),
    "group_of_8": (300, 64, 8, 128, 1, [(1, 97, 300)], 0, 45),
    "group_of_3": (411, 30, 10, 128, 1, [(1, 64, 411)], 0, 30),
    "queries": (90, 64, 8, 128, 4, [(1, 130, 90)], 4, 60),
    "few_stages": (1300, 8, 8, 128, 1, [(1, 1, 1300)], 0, 2),          # fewer stages than wavefronts
    "runs": (1900, 8, 1, 128, 1, [(1, 40, 1900)], 0, 60),
    "d64_queries": (700, 16, 8, 64, 5, [(1, 70, 700)], 5, 50),
}


@pytest.mark.parametrize("cache", ["packed", "paged", "fp8", "paged_fp8_16"])
@pytest.mark.parametrize("rows", [16, 32])
@pytest.mark.parametrize("shape", FOUR_SHAPES)
def test_four_wavefronts(shape, rows, cache):
    B, H, Hkv, D, nq, levels, lo, hi = FOUR_SHAPES[shape]
    print(f"four wavefronts: {shape} rows={rows} {cache}", file=sys.stderr, flush=True)
    w = wl.make_workload(shape, 93, B, H, Hkv, D, levels, lo, hi, nq=nq)
    dw = dev.to_device(w)
    Oref, Lref, call = reference(w, cache)
    options = {hb.HG_OPT_FUSED_KERNEL: 2, hb.HG_OPT_SUFFIX_TILE_ROWS: rows}
    plan = hb.hg_debug_fused_plan(levels, B, nq, H, Hkv, D, dw.max_len, 16 if cache.startswith("paged") else 0, "fp8" in cache, options=options)
    assert (plan["way"], plan["wavefronts"], plan["splits"], plan["column_rows"]) == ("single", 4, 1, rows)
    assert plan["dealt"] == (shape != "runs" or rows == 16 or "fp8" in cache)
    ctx = dev.make_context(dw, parts=32)
    for option, value in options.items():
        ctx.set_option(option, value)
    got = []
    for _ in range(2):
        O = torch.full(dw.lead + (dw.D,), float("nan"), dtype=torch.float32, device="cuda:0")
        L = torch.full(dw.lead, float("nan"), dtype=torch.float32, device="cuda:0")
        call(ctx, dw, O, L)
        got.append((O, L))
    torch.cuda.synchronize()
    check(to_np(got[0][0]), to_np(got[0][1]), Oref, Lref, f"{shape} rows={rows} {cache}")
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    ctx.close()
