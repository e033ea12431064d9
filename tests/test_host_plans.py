"""Host logic of the library, checked without a GPU: the work partition of the persistent shared-block kernel must
cover every (column, stage) position exactly once within the partial results it promises, for any level shape, CU
count and workspace; the suffix planner must respect its limits.  The walk below is the kernel's own rule (mode 0:
team t owns flattened positions [t*quota, (t+1)*quota), part index = team - floor(column * n_c / quota); mode 1: ranges
aligned to the columns), restated in Python."""
import itertools

import numpy as np
import pytest

from paper_2402_05099_amd import binding as hb


def walk(plan):
    """pieces[(column)] = list of (first stage, stages, part index, team) in the order the teams produce them"""
    n_c, ncols, quota = plan["n_c"], plan["ncols"], plan["quota"]
    total = ncols * n_c
    pieces = {}
    nteams = 8 * plan["tpx"]
    for team in range(nteams):
        if plan["mode"] == 2:
            f0, f1, sp = plan["starts"][team], plan["starts"][team + 1], plan["first_part"][team]
        elif plan["mode"] == 0:
            f0, f1 = team * quota, (team + 1) * quota
            sp = team - (f0 // n_c * n_c) // quota
        elif ncols <= nteams:
            c = team * ncols // nteams
            tf = -(-c * nteams // ncols)
            nt = -(-(c + 1) * nteams // ncols) - tf
            sp = team - tf
            f0, f1 = c * n_c + sp * n_c // nt, c * n_c + (sp + 1) * n_c // nt
        else:
            f0, f1 = team * ncols // nteams * n_c, (team + 1) * ncols // nteams * n_c
            sp = 0
        f0, f1 = min(f0, total), min(f1, total)
        c, k0 = divmod(f0, n_c) if f0 < f1 else (0, 0)
        while f0 < f1:
            ln = min(n_c - k0, f1 - f0)
            pieces.setdefault(c, []).append((k0, ln, sp, team))
            f0 += ln
            c += 1
            k0 = 0
            sp = 0          # a later piece of the same team starts its column
    return pieces


SHAPES = [
    # n_blocks, max_rows, max_seqs, Hkv, rows_per_seq
    (1, 16384, 1024, 40, 1), (1, 4096, 512, 8, 8), (1, 2048, 256, 40, 1), (16, 512, 128, 40, 1), (1, 1024, 2048, 40, 1),
    (1, 16384, 1024, 1, 8), (3, 77, 300, 2, 4), (1, 1, 129, 1, 1), (1, 33, 257, 3, 1), (5, 1000, 9000, 4, 2), (1, 31, 40000, 1, 1),
    (2, 100000, 130, 8, 1), (7, 65, 200, 5, 6),
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("slots", [1, 3, 4, 12, 20, 32])
@pytest.mark.parametrize("max_parts", [1, 2, 3, 24, 64])
@pytest.mark.parametrize("D", [128, 64])
def test_wide_plan_covers_every_stage_once(shape, slots, max_parts, D):
    n_blocks, max_rows, max_seqs, Hkv, rps = shape
    plan = hb.hg_debug_wide_plan(n_blocks, max_rows, max_seqs, Hkv, rps, max_parts, slots, D)
    assert plan is not None, "one part per row always fits"
    rows = max_seqs * rps
    mtiles = -(-rows // 256)
    assert plan["n_c"] == -(-max_rows // (32 if D == 128 else 64))      # a stage is 8 KiB of K at either head dimension
    assert plan["rowgroups"] * plan["T"] >= mtiles and (plan["rowgroups"] - 1) * plan["T"] < mtiles
    assert plan["T"] <= plan["slots"] == slots and plan["tpx"] == slots // plan["T"] >= 1
    assert plan["ncols"] == n_blocks * Hkv * plan["rowgroups"]
    assert 1 <= plan["nparts"] <= max_parts
    pieces = walk(plan)
    assert sorted(pieces) == list(range(plan["ncols"])), "every column is visited"
    for c, ps in pieces.items():
        ps.sort()
        assert ps[0][0] == 0 and sum(p[1] for p in ps) == plan["n_c"], "the pieces of a column tile its stages"
        for (k0, ln, _, _), (k1, _, _, _) in zip(ps, ps[1:]):
            assert k0 + ln == k1
        assert [p[2] for p in ps] == list(range(len(ps))), "part indices count the pieces of the column from 0"
        assert len(ps) <= plan["nparts"]
    # the teams that exist can take the whole space
    if plan["mode"] == 0:
        assert 8 * plan["tpx"] * plan["quota"] >= plan["ncols"] * plan["n_c"]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("slots", [1, 3, 5, 12, 20, 32])
@pytest.mark.parametrize("max_parts", [1, 3, 24])
def test_wide_teams_walk_the_ranges_of_the_plan(shape, slots, max_parts):
    """The kernel finds its range with multiplications by numbers from the host: what it computes, for every team, against whole-number divisions here."""
    n_blocks, max_rows, max_seqs, Hkv, rps = shape
    args = (n_blocks, max_rows, max_seqs, Hkv, rps, max_parts, slots, 128)
    plan = hb.hg_debug_wide_plan(*args)
    n_c, ncols, nteams, quota = plan["n_c"], plan["ncols"], 8 * plan["tpx"], plan["quota"]
    for team in range(nteams):
        if plan["mode"] == 2:
            want = plan["starts"][team], plan["starts"][team + 1], plan["first_part"][team]
        elif plan["mode"] == 0:
            want = team * quota, min((team + 1) * quota, n_c * ncols), team - team * quota // n_c * n_c // quota
        elif ncols <= nteams:
            c = team * ncols // nteams
            first = -(-c * nteams // ncols)
            n = -(-(c + 1) * nteams // ncols) - first
            want = c * n_c + (team - first) * n_c // n, c * n_c + (team - first + 1) * n_c // n, team - first
        else:
            want = team * ncols // nteams * n_c, (team + 1) * ncols // nteams * n_c, 0
        assert hb.hg_debug_wide_team(*args, team) == (want if want[0] < want[1] else None), (plan, team)
    assert hb.hg_debug_wide_team(*args, nteams) is None


@pytest.mark.parametrize("slots", [1, 5, 8, 16, 24, 28, 31, 32])
def test_item_runs_cover_every_item_once(slots):
    """Runs of the combined launch: together they hold every item once, a workgroup that starts with a run finds one where there are items for it, and runs are short
    where first runs alone would leave wavefronts without an item."""
    starters = 256 if slots == 32 else 256 - 8 * slots
    for items in sorted({1, 2, 7, starters - 1, starters, starters + 1, 2 * starters - 1, 2 * starters, 4 * starters - 1, 4 * starters, 7 * starters + 3, 8 * starters - 1,
                         8 * starters, 8 * starters + 1, 1023, 1024, 1025, 2048, 2100, 1024 + 8 * starters - 1, 1024 + 8 * starters, 40960, 2**30 - 1} - {0}):
        r = hb.hg_debug_item_runs(items, slots)
        assert r["starters"] == starters and 1 <= r["long_run"] <= 8 and r["tail_run"] in (1, 2)
        assert 0 < r["long_runs"] <= r["runs"] and r["long_runs"] * r["long_run"] <= items
        tail = items - r["long_runs"] * r["long_run"]
        assert (r["runs"] - r["long_runs"] - 1) * r["tail_run"] < tail <= (r["runs"] - r["long_runs"]) * r["tail_run"] or (tail == 0 and r["runs"] == r["long_runs"])
        assert r["runs"] >= min(items, starters)
        if items >= 8 * starters:
            assert r["long_run"] == 8                               # an item for every wavefront at the start
            assert tail <= max(1024 + 7, items - 8 * starters)
        elif items >= starters:
            assert r["long_run"] == items // starters and r["long_runs"] >= starters
        else:
            assert r["long_run"] == 1 and r["long_runs"] == items
    assert hb.hg_debug_item_runs(0, slots) is None and hb.hg_debug_item_runs(2**30, slots) is None and hb.hg_debug_item_runs(5, 33) is None


def test_wide_plan_aligns_short_pieces_to_columns():
    """Config 2's shape (40 columns of 64 stages on 256 teams): ranges of 10 stages would cut 32 teams' ranges at a
    column boundary (two pieces, each with its fixed price); aligned ranges give every team one piece of 9..11 stages."""
    plan = hb.hg_debug_wide_plan(1, 2048, 256, 40, 1, 24, 32)
    assert plan["mode"] == 1 and plan["nparts"] == 7
    pieces = walk(plan)
    per_team = {}
    for c, ps in pieces.items():
        for (k0, ln, sp, team) in ps:
            per_team.setdefault(team, []).append(ln)
    assert all(len(v) == 1 for v in per_team.values()) and len(per_team) == 256
    assert max(v[0] for v in per_team.values()) == 11 and min(v[0] for v in per_team.values()) == 9


def test_wide_plan_gives_ranges_of_equal_cost():
    """Config 3 at 16K keys (40 columns of 512 stages on 64 teams): equal ranges of 320 stages put a column boundary into
    every second team's range.  Ranges of equal cost, a boundary counting as nine stages: 325 stages without a boundary,
    316 with one (321 for a team that ends its column), every (column, stage) still covered once, three parts at most."""
    plan = hb.hg_debug_wide_plan(1, 16384, 1024, 40, 1, 24, 32)
    assert plan["mode"] == 2 and plan["nparts"] == 3 and plan["quota"] == 325
    starts = plan["starts"]
    assert starts[0] == 0 and starts[-1] == 40 * 512 and all(a <= b for a, b in zip(starts, starts[1:]))
    for t in range(64):
        f0, f1 = starts[t], starts[t + 1]
        inner = (f1 - 1) // 512 - f0 // 512
        assert inner <= 1 and (f1 - f0) + 9 * inner <= 325
        assert (f1 - f0) + 9 * inner >= 321                      # nobody is short of work either
    # when every team has a boundary (or none has) the equal ranges stay: config 5's root, config 4
    assert hb.hg_debug_wide_plan(1, 1024, 2048, 40, 1, 24, 32)["mode"] == 0
    assert hb.hg_debug_wide_plan(1, 4096, 512, 8, 8, 24, 32)["mode"] == 0


@pytest.mark.parametrize("max_rows,max_seqs,Hkv,rps,slots,groups,tiles", [
    (395, 563, 2, 32, 28, 4, 18), (389, 168, 8, 32, 28, 1, 21), (16384, 1024, 1, 8, 28, 8, 4),      # short blocks; ends inside ranges
    (4096, 512, 8, 8, 16, 1, 16), (253, 267, 8, 8, 4, 5, 2), (16384, 1024, 40, 1, 20, 1, 4),         # as the products alone decide
])
def test_wide_plan_counts_pieces_when_it_groups_rows(max_rows, max_seqs, Hkv, rps, slots, groups, tiles):
    plan = hb.hg_debug_wide_plan(1, max_rows, max_seqs, Hkv, rps, 24, slots)
    assert (plan["rowgroups"], plan["T"]) == (groups, tiles)
    assert (plan["rowgroups"] - 1) * plan["T"] < -(-max_seqs * rps // 256)
    for ps in walk(plan).values():
        assert sum(p[1] for p in ps) == plan["n_c"] and sorted(p[2] for p in ps) == list(range(len(ps)))


def test_wide_plan_rejects_what_it_cannot_run():
    assert hb.hg_debug_wide_plan(1, 0, 100, 1, 1, 4, 32) is None      # no keys
    assert hb.hg_debug_wide_plan(1, 100, 100, 1, 1, 0, 32) is None     # no room for a result
    assert hb.hg_debug_wide_plan(1, 100, 100, 1, 1, 4, 33) is None     # more CUs per XCD than there are
    assert hb.hg_debug_wide_plan(1, 100, 100, 1, 1, 4, 0) is None
    assert hb.hg_debug_wide_plan(1, 100, 100, 1, 1, 4, 32, 96) is None  # head dimensions other than 64 and 128


@pytest.mark.parametrize("B,nq,Hq,Hkv,D,max_len,ps", [
    (1024, 1, 40, 40, 128, 128, 0), (512, 1, 64, 8, 128, 512, 0), (512, 1, 64, 8, 128, 512, 16), (4, 1, 4, 4, 64, 16, 0),
    (1024, 4, 40, 40, 128, 128, 0), (2048, 1, 40, 40, 128, 64, 0), (3, 1, 8, 1, 128, 5000, 0), (256, 1, 40, 40, 128, 4096, 16),
    (1, 1, 1, 1, 64, 1, 0), (7, 6, 8, 2, 64, 300, 32), (512, 2, 16, 16, 128, 512, 0), (512, 1, 24, 8, 128, 100, 0),
    (512, 1, 16, 8, 128, 512, 0), (512, 1, 16, 8, 128, 128, 0), (512, 1, 16, 8, 128, 256, 16), (64, 1, 32, 32, 128, 383, 0),
    (64, 1, 32, 32, 128, 384, 0),
])
def test_suffix_plan_limits(B, nq, Hq, Hkv, D, max_len, ps):
    p = hb.hg_debug_suffix_plan(B, nq, Hq, Hkv, D, max_len, ps)
    assert p is not None
    assert p["chunk"] % 32 == 0 and p["chunk"] >= 32
    assert p["nchunks"] * p["chunk"] >= max_len and (p["nchunks"] - 1) * p["chunk"] < max(max_len, 1)
    G = Hq // Hkv
    several = nq >= 2 or G >= 3 or (G == 2 and max_len >= 256) or (D == 128 and max_len >= 384)   # ... or long rows to stream
    assert p["mfma"] == int(several), "matrix cores when a KV head serves several rows of a sequence"
    assert G % p["gt"] == 0 and p["gt"] in (1, 2, 4, 8)
    if ps and not p["mfma"]:
        assert p["chunk"] <= 32 * ps, "a vector-ALU work item covers at most 32 pages"


def test_suffix_plan_rejects_bad_arguments():
    assert hb.hg_debug_suffix_plan(4, 1, 6, 4, 128, 10) is None     # Hq not a multiple of Hkv
    assert hb.hg_debug_suffix_plan(4, 1, 4, 4, 96, 10) is None      # unsupported head dimension
    assert hb.hg_debug_suffix_plan(0, 1, 4, 4, 128, 10) is None


# ---- which way a fused call runs (hg_debug_fused_plan) ------------------------------------------------------------------------


def test_fused_plan_names_the_way():
    plan = hb.hg_debug_fused_plan
    assert plan([(1, 128, 4)], 4, 1, 4, 4, 64, 16)["way"] == "single"
    big = plan([(1, 16384, 1024)], 1024, 1, 40, 40, 128, 128)
    assert big["way"] == "combined" and big["wide_levels"] == 1 and big["mfma"] == 0 and 4 <= big["slots"] <= 32
    assert plan([(1, 4096, 512)], 512, 1, 64, 8, 128, 512)["mfma"] == 1
    assert plan([(1, 16384, 1024)], 1024, 1, 40, 40, 128, 128, options={hb.HG_OPT_OVERLAP: 1})["way"] == "one_stream"
    assert plan([(1, 16384, 1024)], 1024, 1, 40, 40, 128, 128, options={hb.HG_OPT_OVERLAP: 2})["way"] == "two_streams"
    assert plan([(1, 0, 4)], 4, 1, 4, 4, 64, 0, options={hb.HG_OPT_FUSED_KERNEL: 1}, workspace_bytes=1 << 20)["way"] == "fill"
    assert plan([(1, 16384, 1024)], 1024, 1, 40, 40, 128, 128, workspace_bytes=0) == hb.HG_ERR_WORKSPACE
    assert plan([], 4, 1, 6, 4, 128, 10) == hb.HG_ERR_UNSUPPORTED
    assert plan([], 0, 1, 4, 4, 128, 10) == hb.HG_ERR_INVALID_ARG
    assert plan([], 4, 1, 4, 4, 128, 10, options={hb.HG_OPT_STAGE_TIMING: 1}) == hb.HG_ERR_INVALID_ARG


# small calls on packed rows: (levels, B, nq, Hq, Hkv, D, max_len)
OWN_MEMORY = [
    ([(1, 128, 4)], 4, 1, 4, 4, 64, 16), ([(1, 515, 45)], 45, 1, 16, 2, 128, 150), ([(1, 1024, 256)], 256, 1, 8, 1, 128, 128),
    ([(1, 441, 72)], 72, 1, 32, 8, 128, 233), ([(1, 1509, 16)], 16, 2, 64, 8, 128, 217), ([(1, 656, 37), (10, 302, 4)], 37, 2, 40, 40, 128, 28),
    ([(13, 840, 4)], 48, 2, 8, 1, 64, 183), ([(1, 927, 265)], 265, 1, 32, 8, 128, 18), ([(1, 211, 1808)], 1808, 2, 8, 1, 128, 21),
    ([(1, 189, 773)], 773, 4, 16, 2, 128, 30), ([(1, 1477, 357), (7, 131, 51)], 357, 1, 40, 40, 128, 92),
    ([], 4, 1, 16, 2, 64, 178), ([], 360, 2, 64, 8, 128, 33), ([], 395, 1, 64, 8, 64, 38), ([], 6, 1, 40, 40, 128, 23),
]


@pytest.mark.parametrize("shape", OWN_MEMORY, ids=str)
def test_small_packed_calls_share_no_memory(shape):
    """One workgroup per column (or the suffix kernel straight to the outputs), whatever the workspace: such calls are accepted
    without one and may be in flight side by side."""
    levels, B, nq, Hq, Hkv, D, max_len = shape
    plans = [hb.hg_debug_fused_plan(levels, B, nq, Hq, Hkv, D, max_len, workspace_bytes=n) for n in (0, 1 << 20, 1 << 34)]
    assert plans[0] == plans[1] == plans[2], plans
    if levels or plans[0]["way"] == "single":
        assert plans[0]["way"] == "single" and plans[0]["splits"] == 1, plans[0]
    else:
        assert plans[0]["way"] == "one_stream" and plans[0]["parts"] == 1
    # the caller's explicit single launch is such a call at any size
    big = hb.hg_debug_fused_plan([(1, 9001, 3)], 3, 1, 4, 1, 128, 70, options={hb.HG_OPT_FUSED_KERNEL: 2})
    assert big["way"] == "single" and big["splits"] == 1


@pytest.mark.parametrize("page,fp8", [(16, False), (0, True), (32, True), (0, False)], ids=["paged", "fp8", "paged_fp8", "packed"])
def test_workspace_decides_whether_a_call_is_accepted(page, fp8):
    """One partial result per shared level and one for the suffix (more where the vector-ALU kernel reads many pages): a call
    that does not find that room is refused however it would run.  (Small packed calls and an explicit single launch need none.)"""
    def plan(levels, B, Hq, Hkv, D, max_len, parts, **kw):
        return hb.hg_debug_fused_plan(levels, B, 1, Hq, Hkv, D, max_len, page, fp8, hb.hg_workspace_bytes(B, Hq, D, parts), **kw)

    shape = ([(1, 9001, 3)], 3, 4, 1, 128, 70) if not (page or fp8) else ([(1, 206, 72)], 72, 32, 8, 128, 40)
    for parts in (0, 1):
        assert plan(*shape, parts) == hb.HG_ERR_WORKSPACE
    assert isinstance(plan(*shape, 2), dict) and plan(*shape, 32)["way"] == "single"
    assert plan(*shape, 0, options={hb.HG_OPT_FUSED_KERNEL: 2})["way"] == "single"
    if page:
        long = ([(1, 60, 2)], 2, 2, 2, 64, 100 * page)      # four items of at most 32 pages each
        assert plan(*long, 4) == hb.HG_ERR_WORKSPACE
        assert plan(*long, 5)["way"] in ("single", "one_stream", "two_streams")


@pytest.mark.parametrize("options", [{}, {hb.HG_OPT_PREFIX_KERNEL: 1}, {hb.HG_OPT_OVERLAP: 1}, {hb.HG_OPT_OVERLAP: 2}], ids=str)
@pytest.mark.parametrize("levels", [[], [(1, 4000, 64)], [(1, 900, 64), (16, 30, 4)]], ids=str)
def test_separate_kernels_are_planned_for_themselves(levels, options):
    """Work items and CUs chosen for the combined launch apply to it only: a call that runs separate kernels (no level of more than
    128 query rows, or an option that rules the combined launch out) cuts its suffix as the suffix call does, and one whose
    options only rule out overlap keeps the whole chip for its shared blocks."""
    options = {hb.HG_OPT_FUSED_KERNEL: 1, **options}
    for B, nq, Hq, Hkv, D, max_len in [(64, 1, 16, 8, 128, 512), (64, 2, 8, 8, 128, 1000), (64, 1, 8, 8, 64, 700)]:
        plan = hb.hg_debug_fused_plan(levels, B, nq, Hq, Hkv, D, max_len, options=options)
        if hb.HG_OPT_PREFIX_KERNEL in options:
            assert plan["way"] != "combined" and plan["slots"] == 0
        elif not levels or (B * nq * Hq // Hkv <= 128):
            assert plan["way"] in ("one_stream", "two_streams")
        if plan["way"] == "combined":
            continue
        alone = hb.hg_debug_suffix_plan(B, nq, Hq, Hkv, D, max_len)
        assert (plan["chunk"], plan["nchunks"]) == (alone["chunk"], alone["nchunks"]), (plan, alone)


@pytest.mark.parametrize("shape", [([(1, 5766, 576)], 576, 128, 23, False), ([(1, 3028, 867)], 867, 64, 16, False), ([(1, 11315, 179), (15, 91, 12)], 179, 128, 23, False),
                                   ([(1, 190, 965)], 965, 64, 29, True), ([(1, 79, 832)], 832, 64, 71, True), ([(1, 2268, 1802)], 1802, 128, 36, True)], ids=str)
def test_short_suffixes_of_one_row_do_not_join_the_shared_block(shape):
    """One query row per KV head and few rows: separate kernels (the combined launch took up to 24 % longer on calls like these), or, over codes at
    D = 64 and few keys, the single launch (64 -> 38 and 69 -> 56 us)."""
    levels, B, D, max_len, fp8 = shape
    separate = hb.hg_debug_fused_plan(levels, B, 1, 40, 40, D, max_len, 0, fp8, options={hb.HG_OPT_FUSED_KERNEL: 1})
    assert separate["way"] in ("one_stream", "two_streams")
    assert hb.hg_debug_fused_plan(levels, B, 1, 40, 40, D, max_len, 0, fp8)["way"] == ("single" if fp8 and D == 64 else separate["way"])
    assert hb.hg_debug_fused_plan(levels, B, 1, 40, 40, D, 300, 0, fp8)["way"] == "combined"
    assert hb.hg_debug_fused_plan(levels, B, 1, 40, 40, D, max_len, 0, fp8, options={hb.HG_OPT_FUSED_KERNEL: 1, hb.HG_OPT_WIDE_SLOTS: 16})["way"] == "combined"


@pytest.mark.parametrize("shape", [([(1, 5204, 104)], 104, 40, 26, 0), ([(1, 7000, 120)], 120, 40, 30, 0), ([(1, 12000, 100)], 100, 40, 40, 0), ([(1, 6000, 128)], 128, 40, 300, 0)], ids=str)
def test_small_calls_on_separate_kernels_where_those_are_faster(shape):
    """8-bit rows, one query row per KV head: the single launch took 8 to 56 % longer on these (on a few rows, or a few keys, it is the faster)."""
    levels, B, H, max_len, page = shape
    assert hb.hg_debug_fused_plan(levels, B, 1, H, H, 128, max_len, page, True)["way"] in ("one_stream", "two_streams")
    assert hb.hg_debug_fused_plan([(1, 269, 5)], 5, 1, 40, 40, 128, 37, page, True)["way"] == "single"
    assert hb.hg_debug_fused_plan([(1, 95, 14)], 14, 1, 4, 4, 128, 539)["way"] == "single"      # (long rows: matrix cores; 23 against 29 us)


@pytest.mark.parametrize("shape", [([(1, 76, 1880)], 1880, 4, 128, 29, 16), ([(1, 156, 155)], 155, 40, 128, 41, 0), ([(1, 6705, 323)], 323, 4, 64, 45, 16),
                                   ([(1, 660, 171)], 171, 40, 64, 32, 0), ([(1, 1697, 733)], 733, 4, 64, 73, 0), ([(1, 9424, 330)], 330, 4, 64, 93, 0), ([(1, 583, 9)], 9, 4, 128, 350, 16),
                                   ([(1, 299, 30)], 30, 4, 128, 200, 16), ([(1, 336, 95)], 95, 40, 128, 39, 0), ([(1, 219, 37)], 37, 40, 128, 23, 0), ([(1, 3511, 41)], 41, 40, 128, 31, 0)], ids=str)
def test_small_calls_in_one_launch_where_that_is_faster(shape):
    """8-bit rows, one query row per KV head, a shared block for the persistent kernel, D = 64 or few sequences: 20 to 60 % faster in the single launch.  The
    last four, small blocks on kernels of their own: 18.7 -> 10.2, 25.2 -> 13.9, 17.6 -> 11.2 and 28.7 -> 22.6 us."""
    levels, B, H, D, max_len, page = shape
    assert hb.hg_debug_fused_plan(levels, B, 1, H, H, D, max_len, page, True)["way"] == "single"


# a suffix alone, one work item per row of the matrix-core kernel: (B, nq, Hq, Hkv, max_len, page, codes)
@pytest.mark.parametrize("shape,way", [
    ((607, 4, 8, 1, 26, 0, False), "one_stream"), ((547, 2, 64, 8, 383, 16, False), "one_stream"), ((822, 2, 8, 1, 62, 32, True), "one_stream"),
    ((123, 4, 64, 8, 22, 0, False), "one_stream"), ((898, 4, 8, 1, 142, 64, True), "one_stream"), ((144, 1, 64, 8, 19, 0, True), "one_stream"),
    ((6, 1, 32, 8, 1, 0, True), "single"), ((16, 1, 8, 1, 20, 16, False), "single"), ((197, 4, 40, 40, 25, 0, False), "single"), ((647, 4, 4, 4, 20, 0, False), "single"), ((416, 1, 32, 8, 34, 0, False), "single"),
], ids=str)
def test_suffixes_alone_go_by_their_work_items(shape, way):
    """Few items, or rows enough to stream, run on the suffix kernel (the single launch took 10 to 60 % longer on the first six), many short items,
    and next to none, in the single launch (the suffix kernel took 1.1 to 2 times as long on the others)."""
    B, nq, Hq, Hkv, max_len, page, codes = shape
    plan = hb.hg_debug_fused_plan([], B, nq, Hq, Hkv, 128, max_len, page, codes)
    assert plan["way"] == way, plan
    if way == "one_stream":
        assert plan["mfma"] == 1 and plan["parts"] == 1


@pytest.mark.parametrize("shape", [([(1, 9973, 185)], 185, 1, 16, 2, 128, 386), ([(1, 9224, 432)], 432, 1, 8, 1, 128, 319), ([(1, 4186, 326)], 326, 1, 16, 2, 128, 298),
                                   ([(1, 6622, 762)], 762, 1, 4, 4, 128, 49), ([(1, 973, 253)], 253, 1, 4, 4, 64, 993)], ids=str)
def test_many_parts_of_the_combined_launch_are_priced(shape):
    """A few columns with many keys: the combined launch cuts them into many parts (it took 1.2 to 1.46 times as long as the single launch on these).
    Where the workspace does not hold them all, their price is not counted."""
    levels, B, nq, Hq, Hkv, D, max_len = shape
    plan = lambda parts, **kw: hb.hg_debug_fused_plan(levels, B, nq, Hq, Hkv, D, max_len, workspace_bytes=hb.hg_workspace_bytes(B * nq, Hq, D, parts), **kw)
    assert plan(24)["way"] == "single"
    other = plan(24, options={hb.HG_OPT_FUSED_KERNEL: 1})
    assert other["way"] == "combined" and other["parts"] > 8
    assert plan(2)["way"] in ("combined", "one_stream", "two_streams")


@pytest.mark.parametrize("shape", [([(1, 3804, 286), (7, 41, 41)], 286, 1, 32, 8, 102, 0, False), ([(1, 7199, 72), (14, 102, 6)], 72, 4, 40, 40, 72, 0, False),
                                   ([(1, 4105, 142), (6, 961, 24)], 142, 1, 32, 8, 334, 0, True), ([(1, 814, 331), (2, 142, 166)], 331, 1, 32, 8, 482, 0, True),
                                   ([(1, 4542, 100), (16, 922, 7)], 100, 1, 40, 40, 105, 64, True)], ids=str)
def test_trees_of_a_few_more_columns_than_cus(shape):
    """Four wavefronts per workgroup with 257 to 511 columns, and codes on the matrix cores: the single launch took 1.2 to 1.6 times as long on these."""
    levels, B, nq, Hq, Hkv, max_len, page, codes = shape
    plan = lambda levels: hb.hg_debug_fused_plan(levels, B, nq, Hq, Hkv, 128, max_len, page, codes, workspace_bytes=hb.hg_workspace_bytes(B * nq, Hq, 128, 24))
    assert plan(levels)["way"] in ("combined", "one_stream", "two_streams")


@pytest.mark.parametrize("shape,wavefronts", [(([(11, 883, 27)], 290, 4, 4, 4, 64, 74, 0, True), 8), (([(1, 977, 35)], 35, 2, 64, 8, 64, 37, 0, True), 8),
                                              (([(1, 312, 100)], 100, 1, 40, 40, 64, 17, 32, True), 8), (([(5, 459, 116)], 577, 1, 8, 1, 64, 74, 16, True), 8),
                                              (([(1, 65, 27)], 27, 2, 64, 8, 64, 18, 0, False), 4), (([(1, 549, 683)], 683, 4, 64, 8, 128, 60, 0, False), 4)], ids=str)
def test_four_wavefronts_where_columns_outnumber_their_places(shape, wavefronts):
    """Up to 256 columns (16 rows of D = 64: 512) run at once in workgroups of eight wavefronts and are the faster so (by a fifth to a third on the first four),
    unless a column has fewer stages than those."""
    levels, B, nq, Hq, Hkv, D, max_len, page, codes = shape
    plan = hb.hg_debug_fused_plan(levels, B, nq, Hq, Hkv, D, max_len, page, codes, workspace_bytes=hb.hg_workspace_bytes(B * nq, Hq, D, 24))
    assert (plan["way"], plan["wavefronts"]) == ("single", wavefronts), plan


def test_options_of_the_separate_kernels_ask_for_them():
    """An option names the kernel it tunes: small calls on paged or 8-bit rows then run that kernel instead of the single launch, items
    per wavefront and splits of the 128-row kernel are not dropped in the combined launch."""
    small = lambda **kw: hb.hg_debug_fused_plan([(1, 206, 72)], 72, 1, 32, 8, 128, 40, 16, **kw)
    assert small()["way"] == "single"
    for option, value in [(hb.HG_OPT_PREFIX_SPLITS, 2), (hb.HG_OPT_SUFFIX_CHUNK, 32), (hb.HG_OPT_OVERLAP, 1), (hb.HG_OPT_PREFIX_KERNEL, 1),
                          (hb.HG_OPT_WIDE_SLOTS, 8), (hb.HG_OPT_SUFFIX_KERNEL, 1), (hb.HG_OPT_SUFFIX_ITEMS_PER_WAVE, 3), (hb.HG_OPT_SUFFIX_TILE_ROWS, 32)]:
        assert small(options={option: value})["way"] != "single", option
    tree = lambda **kw: hb.hg_debug_fused_plan([(1, 1024, 2048), (16, 512, 128)], 2048, 1, 40, 40, 128, 64, **kw)
    assert tree()["way"] == "combined" and tree()["wide_levels"] == 3
    assert tree(options={hb.HG_OPT_PREFIX_SPLITS: 3})["wide_levels"] == 1
    gqa = lambda **kw: hb.hg_debug_fused_plan([(1, 4096, 512)], 512, 1, 64, 8, 128, 512, **kw)
    assert gqa()["way"] == "combined"
    assert gqa(options={hb.HG_OPT_SUFFIX_ITEMS_PER_WAVE: 3})["way"] in ("one_stream", "two_streams")


@pytest.mark.parametrize("shape", [([(1, 2048, 256)], 256, 40, 40, 256, 0, False), ([(1, 253, 267)], 267, 64, 8, 397, 0, True), ([(1, 515, 130)], 130, 32, 8, 665, 16, False)], ids=str)
def test_combined_calls_bound_by_their_suffix_give_the_shared_levels_five_cus(shape):
    """And never fewer, also where the workspace only just holds the parts."""
    levels, B, Hq, Hkv, max_len, page, fp8 = shape
    plan = hb.hg_debug_fused_plan(levels, B, 1, Hq, Hkv, 128, max_len, page, fp8)
    assert (plan["way"], plan["slots"]) == ("combined", 5)
    room = hb.hg_workspace_bytes(B, Hq, 128, plan["parts"])
    assert hb.hg_debug_fused_plan(levels, B, 1, Hq, Hkv, 128, max_len, page, fp8, workspace_bytes=room) == plan
    less = hb.hg_debug_fused_plan(levels, B, 1, Hq, Hkv, 128, max_len, page, fp8, workspace_bytes=hb.hg_workspace_bytes(B, Hq, 128, plan["parts"] - 1))
    assert isinstance(less, int) or less["parts"] < plan["parts"]


@pytest.mark.parametrize("tiles,splits,Hkv", [(1, 1, 1), (3, 7, 40), (65537, 1, 5), (1000003, 1, 40), (46341, 31, 40), (2**20 + 1, 16, 64), (8388593, 32, 8 - 1), (2**31 // 8 - 3, 1, 8)])
def test_divisions_by_numbers_from_the_host(tiles, splits, Hkv):
    """The kernels divide by multiplying with a number from the host; exact for every numerator below 2^31.  Here through the work of
    a workgroup of a single launch, over divisors and numerators up to the limits."""
    n = tiles * splits * Hkv
    rng = np.random.default_rng(3)
    for x in range(8):
        first, end = x * n // 8, (x + 1) * n // 8
        near = [a + d for a in (first, (first + end) // 2, (first // (tiles * splits) + 1) * tiles * splits, end) for d in (-2, -1, 0, 1)]
        for at in sorted({a for a in near + rng.integers(first, max(end, first + 1), 20).tolist() if first <= a < end}):
            kvh, rest = divmod(at, tiles * splits)
            assert hb.hg_debug_single_work(8 * (at - first) + x, tiles, splits, Hkv) == (kvh, *divmod(rest, splits)), at


@pytest.mark.parametrize("tiles,splits,Hkv", [(1, 1, 1), (7, 1, 1), (3, 5, 1), (2, 3, 10), (5, 1, 3), (4, 5, 10), (4, 5, 12), (9, 1, 36), (13, 2, 8), (6, 1, 40), (1, 32, 5)])
def test_single_launch_deals_heads_out_to_the_xcds(tiles, splits, Hkv):
    """Every column and split once, the same number for every XCD, and the workgroups of a KV head side by side: on its share of the
    XCDs (and the two that it may have in common with its neighbours) for any number of heads."""
    grid = -(-tiles * splits * Hkv // 8) * 8
    work = {i: hb.hg_debug_single_work(i, tiles, splits, Hkv) for i in range(grid)}
    got = {w: i % 8 for i, w in work.items() if w}
    assert sorted(got) == [(h, t, s) for h in range(Hkv) for t in range(tiles) for s in range(splits)] and len(got) == sum(w is not None for w in work.values())
    assert hb.hg_debug_single_work(grid, tiles, splits, Hkv) is None
    counts = [sum(x == y for y in got.values()) for x in range(8)]
    assert max(counts) - min(counts) <= 1
    for h in range(Hkv):
        assert len({x for w, x in got.items() if w[0] == h}) <= -(-8 // Hkv) + 1


@pytest.mark.parametrize("shape,way", [
    (([(1, 5000, 216)], 216, 32, 8, 64, 0, True), "combined"), (([(1, 5000, 216)], 216, 32, 8, 128, 0, True), "combined"), (([(1, 5000, 216)], 216, 32, 8, 200, 0, True), "combined"),
    (([(1, 4500, 150)], 150, 32, 8, 100, 0, True), "combined"), (([(1, 5000, 180)], 180, 32, 8, 150, 0, True), "combined"),
    (([(1, 3189, 106)], 106, 32, 8, 475, 16, False), "combined"),
    (([(1, 8192, 64)], 64, 40, 10, 100, 16, False), "single"), (([(1, 10500, 34)], 34, 32, 8, 100, 16, False), "single"), (([(1, 1026, 341)], 341, 32, 8, 20, 0, True), "single"),
], ids=str)
def test_combined_launch_is_priced_beside_the_single_one(shape, way):
    """Many columns that walk one long shared block with a workgroup each (48 against 40 us and the like); fewer, whose blocks several
    workgroups share, stay in the single launch.  Only the workspace may refuse a call, whichever way it would take."""
    levels, B, Hq, Hkv, max_len, page, fp8 = shape
    call = lambda **kw: hb.hg_debug_fused_plan(levels, B, 1, Hq, Hkv, 128, max_len, page, fp8, **kw)      # noqa: E731
    assert call()["way"] == way
    assert call(workspace_bytes=hb.hg_workspace_bytes(B, Hq, 128, 2))["way"] in ("single", "combined")
    assert call(workspace_bytes=hb.hg_workspace_bytes(B, Hq, 128, 1)) == hb.HG_ERR_WORKSPACE


@pytest.mark.parametrize("shape,rows,splits", [
    (([(1, 128, 4)], 4, 1, 4, 4, 64, 16), 16, 1), (([(1, 515, 45)], 45, 1, 16, 2, 128, 150), 16, 1), (([(1, 515, 95)], 95, 2, 16, 2, 128, 60), 16, 1),
    (([(1, 300, 139)], 139, 4, 64, 8, 128, 64), 32, 1),                                             # twice the columns would take two rounds
    (([(1, 3000, 60)], 60, 1, 16, 2, 128, 100, 16), 16, 4), (([(1, 4000, 100)], 100, 1, 32, 8, 128, 60, 16), 32, 2), (([(1, 9000, 20)], 20, 1, 16, 2, 128, 60, 0, True), 16, 12),
], ids=str)
def test_rows_and_workgroups_of_the_single_launch(shape, rows, splits):
    """What the library chooses by itself; a workspace that just holds the results of that many workgroups per column keeps the choice, a byte less does not."""
    levels, B, nq, Hq, Hkv, D = shape[:6]
    plan = hb.hg_debug_fused_plan(*shape)
    assert (plan["way"], plan["column_rows"], plan["splits"]) == ("single", rows, splits)
    if splits > 1:
        cols = -(-B * nq * Hq // Hkv // rows) * Hkv
        room = cols * splits * rows * (D + 2) * 4
        assert hb.hg_debug_fused_plan(*shape, workspace_bytes=room) == plan
        assert hb.hg_debug_fused_plan(*shape, workspace_bytes=room - 1) != plan
    # asked for by option
    for asked in (16, 32):
        forced = hb.hg_debug_fused_plan(*shape, options={hb.HG_OPT_FUSED_KERNEL: 2, hb.HG_OPT_SUFFIX_TILE_ROWS: asked})
        assert (forced["way"], forced["column_rows"]) == ("single", asked)


@pytest.mark.parametrize("shape,dealt", [
    (([(1, 1024, 1024)], 1024, 1, 8, 1, 128, 128), False), (([(1, 1024, 2048)], 2048, 1, 8, 1, 128, 512), False), (([(1, 532, 456)], 456, 1, 16, 2, 128, 184), False),
    (([(1, 4096, 1024)], 1024, 1, 8, 1, 128, 128), True),       # the shared rows are most of the call
    (([(1, 1024, 256)], 256, 1, 8, 1, 128, 512), True),         # 16 rows
    (([(1, 100, 90)], 90, 1, 32, 8, 128, 200), True), (([(1, 300, 1000)], 1000, 1, 8, 1, 64, 300), True),
], ids=str)
def test_stages_of_the_single_launch_in_runs_where_the_suffix_decides(shape, dealt):
    plan = hb.hg_debug_fused_plan(*shape)
    assert (plan["way"], plan["dealt"]) == ("single", dealt)


@pytest.mark.parametrize("shape,way,rows", [
    (([(1, 7171, 109)], 109, 1, 40, 40, 64, 69, 32), "one_stream", None), (([(1, 8192, 112)], 112, 1, 40, 40, 64, 8), "one_stream", None),
    (([(1, 4171, 264)], 264, 1, 32, 8, 64, 207, 64, True), "one_stream", None), (([(1, 2048, 112)], 112, 1, 40, 40, 64, 8), "single", 32),
], ids=str)
def test_two_workgroups_share_a_cu_at_head_dimension_64(shape, way, rows):
    """More than 256 columns take longer than 256 though they all run at a time: 280 columns of 16 rows 37, 66 and 108 us where 160 of 32 rows or
    separate kernels take 30, 41 and 60."""
    plan = hb.hg_debug_fused_plan(*shape)
    assert (plan["way"], plan.get("column_rows")) == (way, rows)


@pytest.mark.parametrize("shape,way", [(([(1, 7168, 109)], 109, 1, 40, 40, 64, 68), "one_stream"), (([(1, 9454, 400)], 400, 1, 16, 16, 128, 20), "one_stream"), (([(1, 8607, 193)], 193, 1, 16, 16, 128, 83, 16), "combined"),
                                       (([(1, 4096, 109)], 109, 1, 40, 40, 64, 32), "single"), (([(1, 9303, 19)], 19, 1, 40, 40, 128, 152), "single")], ids=str)
def test_shared_rows_that_no_cache_holds_leave_the_single_launch(shape, way):
    """Few columns per KV head re-read them for stages that then wait for the HBM: 76 us against 48 on separate kernels, 69 against 49 in the combined launch."""
    assert hb.hg_debug_fused_plan(*shape)["way"] == way
