"""The single launch with several workgroups per 32-row column (they meet through counters and the workspace) and over every
suffix cache: packed, paged, 8-bit, paged 8-bit.  Seeded random trees against the fp64 oracle; every call runs twice in
a row (the first must leave its counters at zero) with the same bits, with and without room for partial results.  (Asked
for by option, packed rows are not split: those cells run one workgroup per column; test_split_launch_of_packed_rows has
the ones that the automatic choice splits.)"""
import ctypes
import sys

import pytest
import torch

import oracle
from oracle import fp8
from paper_2402_05099_amd import binding as hb
from paper_2402_05099_amd import device as dev
from paper_2402_05099_amd import workloads as wl
from parity import check, to_np
from test_gpu_random_shapes import random_workload

pytestmark = pytest.mark.gpu


def reference(w, cache):
    """(O, LSE, caller of the fused entry point) of workload w with its suffix in the given cache."""
    if cache == "packed":
        O, L = oracle.attention(w)
        return O, L, lambda c, dw, o, l: hb.hg_hydragen_attn(c, dw.Q, dw.levels, dw.Ks, dw.Vs, dw.offsets, dw.lengths, dw.max_len, o, l, dw.scale)
    if cache == "paged":
        O, L = oracle.attention(w)
        kv = dev.paged_to_device(wl.make_paged(w, 16))
        return O, L, lambda c, dw, o, l: hb.hg_hydragen_attn_paged(c, dw.Q, dw.levels, kv, dw.lengths, dw.max_len, o, l, dw.scale)
    f8 = wl.make_fp8(w, reserve=2)
    O, L = fp8.suffix_attention_fp8(w.Q, w.Hkv, f8.Ks8, f8.Vs8, f8.k_scale, f8.v_scale, f8.offsets, w.lengths, w.scale)
    if w.levels:
        Op, Lp = oracle.attention(w, suffix=False)
        O, L = oracle.merge([Op, O], [Lp, L])
    if cache == "fp8":
        Ks8, Vs8, off = (torch.from_numpy(x).cuda() for x in (f8.Ks8, f8.Vs8, f8.offsets))
        return O, L, lambda c, dw, o, l: hb.hg_hydragen_attn_fp8(c, dw.Q, dw.levels, Ks8, Vs8, f8.k_scale, f8.v_scale, off, dw.lengths,
                                                                dw.max_len, o, l, dw.scale)
    pg, ks, vs = wl.make_paged_fp8(w, 16 if cache == "paged_fp8_16" else 32)
    kv = hb.PagedKV(K=torch.from_numpy(pg.K).cuda(), V=torch.from_numpy(pg.V).cuda(), page_table=torch.from_numpy(pg.table).cuda(),
                    page_size=pg.page_size, kv_format=hb.HG_KV_E4M3, k_scale=ks, v_scale=vs)
    return O, L, lambda c, dw, o, l: hb.hg_hydragen_attn_paged(c, dw.Q, dw.levels, kv, dw.lengths, dw.max_len, o, l, dw.scale)


def calls(w, cache, what):
    if w.max_len == 0:
        pytest.skip("no suffix rows: the caches do not differ")
    dw = dev.to_device(w)
    Oref, Lref, call = reference(w, cache)
    for parts in (32, 0):                     # room for partial results (split columns), none (one workgroup per column)
        ctx = dev.make_context(dw, parts=parts) if parts else hb.Context(0, 0)
        ctx.set_option(hb.HG_OPT_FUSED_KERNEL, 2)
        got = []
        for _ in range(2):
            O = torch.full(dw.lead + (dw.D,), float("nan"), dtype=torch.float32, device="cuda:0")
            L = torch.full(dw.lead, float("nan"), dtype=torch.float32, device="cuda:0")
            call(ctx, dw, O, L)
            got.append((O, L))
        torch.cuda.synchronize()
        check(to_np(got[0][0]), to_np(got[0][1]), Oref, Lref, f"{what} parts={parts}")
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), f"{what}: the second call differs"
        ctx.close()


@pytest.mark.parametrize("cache", ["packed", "paged", "fp8", "paged_fp8"])
@pytest.mark.parametrize("seed", range(16))
def test_split_launch_random_trees(seed, cache):
    w = random_workload(seed)
    print(f"split launch: random shape {seed} {cache}: B={w.B} Hq={w.Hq} Hkv={w.Hkv} D={w.D} nq={w.nq} "
          f"levels={[(l.Gn, l.max_rows) for l in w.levels]} max_len={w.max_len}", file=sys.stderr, flush=True)
    calls(w, cache, f"random {seed} {cache}")


@pytest.mark.parametrize("shape", [(3, 4, 1, 128, 9001, 70), (3, 4, 1, 64, 9001, 70), (7, 16, 2, 128, 5000, 33), (40, 16, 2, 64, 4100, 1)], ids=str)
def test_split_launch_of_packed_rows(shape):
    """Packed rows and a long block: several workgroups per column by the automatic choice."""
    B, Hq, Hkv, D, P, hi = shape
    print(f"split launch: packed rows {shape}", file=sys.stderr, flush=True)
    w = wl.make_workload("packed split", 47, B, Hq, Hkv, D, [(1, P, B)], 1, hi)
    dw = dev.to_device(w)
    Oref, Lref, call = reference(w, "packed")
    plan = hb.hg_debug_fused_plan([(1, P, B)], B, 1, Hq, Hkv, D, dw.max_len, workspace_bytes=hb.hg_workspace_bytes(B, Hq, D, 32))
    assert plan["way"] == "single" and plan["splits"] > 1, plan
    ctx = dev.make_context(dw, parts=32)
    ctx.set_option(hb.HG_OPT_FUSED_KERNEL, 0)
    got = []
    for _ in range(2):
        O = torch.full(dw.lead + (D,), float("nan"), dtype=torch.float32, device="cuda:0")
        L = torch.full(dw.lead, float("nan"), dtype=torch.float32, device="cuda:0")
        call(ctx, dw, O, L)
        got.append((O, L))
    torch.cuda.synchronize()
    check(to_np(got[0][0]), to_np(got[0][1]), Oref, Lref, f"packed split {shape}")
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    ctx.close()


@pytest.mark.parametrize("cache", ["packed", "paged_fp8"])
@pytest.mark.parametrize("D", [64, 128])
def test_split_launch_long_block(D, cache):
    """One column, a block long enough for the largest number of workgroups per column."""
    print(f"split launch: long block D={D} {cache}", file=sys.stderr, flush=True)
    calls(wl.make_workload("long", 41, 3, 4, 1, D, [(1, 9001, 3)], 1, 70), cache, f"long block D={D} {cache}")


@pytest.mark.parametrize("P", [6000, 9001, 12000, 30000, 60000])
@pytest.mark.parametrize("option", [0, 2])
@pytest.mark.parametrize("D", [64, 128])
def test_split_launch_many_partial_results(D, option, P):
    """The last workgroup of a column reads up to 16 (columns of 16 rows, or D = 64) or 8 results at a time: fewer, as many, one more
    and several times as many, over empty suffixes (sequence 1 has none)."""
    w = wl.make_workload("many parts", 48, 3, 4, 1, D, [(1, P, 3)], 1, 70)
    w.lengths[1] = 0
    kv = dev.paged_to_device(wl.make_paged(w, 16))
    dw = dev.to_device(w)
    plan = hb.hg_debug_fused_plan([(1, P, 3)], 3, 1, 4, 1, D, dw.max_len, 16, options={hb.HG_OPT_FUSED_KERNEL: option})
    assert plan["way"] == "single" and plan["splits"] > 4, plan
    print(f"split launch: D={D} option {option}: {plan['splits']} results of {plan['column_rows']} rows", file=sys.stderr, flush=True)
    ctx = dev.make_context(dw, parts=64)
    ctx.set_option(hb.HG_OPT_FUSED_KERNEL, option)
    O = torch.full(dw.lead + (D,), float("nan"), dtype=torch.float32, device="cuda:0")
    L = torch.full(dw.lead, float("nan"), dtype=torch.float32, device="cuda:0")
    hb.hg_hydragen_attn_paged(ctx, dw.Q, dw.levels, kv, dw.lengths, dw.max_len, O, L, dw.scale)
    torch.cuda.synchronize()
    check(to_np(O), to_np(L), *oracle.attention(w), f"{plan['splits']} results")
    ctx.close()


def test_one_context_alternates_between_ways_and_splits():
    """Split single launches with different numbers of workgroups per column, and combined launches, take turns on one context
    and its counters, some of them captured: every call leaves the counters as the next one needs them."""
    small = [wl.make_workload("s1", 42, 5, 8, 1, 128, [(1, 6000, 5)], 1, 30), wl.make_workload("s2", 43, 60, 8, 2, 128, [(1, 900, 60)], 1, 30),
             wl.make_workload("s3", 44, 20, 8, 4, 128, [(1, 400, 20)], 1, 90)]
    big = wl.make_workload("big", 45, 300, 8, 1, 128, [(1, 200, 300)], 1, 40)
    work = []
    splits = set()
    for w in small + [big]:
        kv = dev.paged_to_device(wl.make_paged(w, 16))
        dw = dev.to_device(w)
        option = 1 if w is big else 2
        rps = w.nq * w.Hq // w.Hkv
        plan = hb.hg_debug_fused_plan([(l.Gn, l.max_rows, w.B) for l in w.levels], w.B, 1, w.Hq, w.Hkv, w.D, dw.max_len, 16,
                                      options={hb.HG_OPT_FUSED_KERNEL: option})
        assert plan["way"] == ("combined" if w is big else "single"), plan
        splits.add(plan["splits"])
        work.append((dw, kv, option, *oracle.attention(w)))
    assert len(splits) == 4, splits
    ctx = hb.Context(0, hb.hg_workspace_bytes(300, 8, 128, 32))

    def call(dw, kv, option):
        O = torch.full(dw.lead + (dw.D,), float("nan"), dtype=torch.float32, device="cuda:0")
        L = torch.full(dw.lead, float("nan"), dtype=torch.float32, device="cuda:0")
        ctx.set_option(hb.HG_OPT_FUSED_KERNEL, option)
        hb.hg_hydragen_attn_paged(ctx, dw.Q, dw.levels, kv, dw.lengths, dw.max_len, O, L, dw.scale)
        return O, L

    first = []
    for dw, kv, option, Oref, Lref in work:
        print(f"ways in turn: B={dw.B} option {option}", file=sys.stderr, flush=True)
        O, L = call(dw, kv, option)
        torch.cuda.synchronize()
        check(to_np(O), to_np(L), Oref, Lref, f"B={dw.B}")
        first.append((O, L))
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ctx.set_stream(side)
        captured = [call(dw, kv, option) for dw, kv, option, _, _ in work]
    ctx.set_stream(None)
    for turn in range(12):
        i = (turn * 5 + turn // 3) % 4
        O, L = call(*work[i][:3])
        torch.cuda.synchronize()
        assert torch.equal(O, first[i][0]) and torch.equal(L, first[i][1]), f"turn {turn}"
        if turn % 4 == 1:
            graph.replay()
            torch.cuda.synchronize()
            for (o, l), (fo, fl) in zip(captured, first):
                assert torch.equal(o, fo) and torch.equal(l, fl), f"replay at turn {turn}"
    ctx.close()


def test_contexts_beyond_the_counter_slots_while_a_stream_is_captured():
    """Counter slots come back from closed contexts without anybody waiting: more contexts than there are slots are created, used
    and closed while their calls are in flight, the last ones while a stream is being captured.  Every call has the bits of
    the first (a context without counters would not split its columns), and so has the graph replayed at the end, long after its
    context is gone."""
    print("split launch: 1100 contexts", file=sys.stderr, flush=True)
    w = wl.make_workload("slots", 46, 5, 8, 1, 128, [(1, 6000, 5)], 1, 30)
    kv = dev.paged_to_device(wl.make_paged(w, 16))
    dw = dev.to_device(w)
    ws = torch.empty(hb.hg_workspace_bytes(5, 8, 128, 32), dtype=torch.uint8, device="cuda:0")

    def call(stream=None):
        ctx = hb.Context(0, 0, stream=stream)      # (a context per call on one workspace: the calls are ordered on one stream)
        ctx.close()
        h = ctypes.c_void_p()
        hb._check(hb.lib().hg_create(ctypes.byref(h), 0, ctypes.c_void_p(ctx._stream_handle(stream)), hb._p(ws), ws.numel()), "hg_create")
        ctx.h = h
        ctx.set_option(hb.HG_OPT_FUSED_KERNEL, 2)
        O = torch.empty(dw.lead + (dw.D,), dtype=torch.float32, device="cuda:0")
        L = torch.empty(dw.lead, dtype=torch.float32, device="cuda:0")
        hb.hg_hydragen_attn_paged(ctx, dw.Q, dw.levels, kv, dw.lengths, dw.max_len, O, L, dw.scale)
        ctx.close()
        return O, L

    first = call()
    torch.cuda.synchronize()
    check(to_np(first[0]), to_np(first[1]), *oracle.attention(w), "first context")
    for i in range(1100):
        O, L = call()
        if i % 100 == 0:
            torch.cuda.synchronize()
            assert torch.equal(O, first[0]) and torch.equal(L, first[1]), f"context {i}"
    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for _ in range(1100):
            hb.Context(0, 0, stream=side).close()
        captured = [call(side) for _ in range(3)]
    for i in range(20):
        O, L = call()
        torch.cuda.synchronize()
        assert torch.equal(O, first[0]) and torch.equal(L, first[1]), f"context {i} after the capture"
        if i % 5 == 0:
            for o, l in captured:
                o.fill_(float("nan"))
                l.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for o, l in captured:
                assert torch.equal(o, first[0]) and torch.equal(l, first[1]), f"replay {i}"
