"""The native marshalling of the decode-step calls (csrc/marshal.cpp): what the checks in Python refuse it never passes on,
what they accept works through either, with the same results."""
import types
import warnings

import pytest
import torch

from paper_2402_05099_amd import binding as hb


def test_what_is_not_plain_is_left_to_python():
    """Host tensors, tensors of a transform, wrong counts and other objects: None, and no exception left behind."""
    m = hb.native()
    q = torch.zeros(2, 2, 64, dtype=torch.bfloat16)
    ctx = types.SimpleNamespace(h=hb.ctypes.c_void_p(1))
    assert m.attn(ctx, q, [], q, q, q, q, 1, q, q, 0.0) is None
    assert m.attn() is None and m.append(1, 2) is None
    assert m.attn_paged(*[object()] * 9) is None
    got = []
    torch.vmap(lambda x: got.append(m.append(ctx, x, x, x, x, x, x, 1)) or x)(q)
    assert got == [None]


def test_refusals_are_those_of_python():
    q = torch.zeros(2, 2, 64, dtype=torch.bfloat16)
    n = torch.zeros(2, dtype=torch.int32)
    kv = hb.PagedKV(q, q, n, 16)
    for call in (lambda: hb.hg_hydragen_attn(None, q, [], q, q, n, n, 1, q), lambda: hb.hg_kv_append(None, q, q, q, q, n, n, 1),
                 lambda: hb.hg_kv_append_fp8(None, q, q, q, q, 1.0, 1.0, n, n, 1), lambda: hb.hg_kv_append_paged(None, q, q, kv, n, 1)):
        with pytest.raises(TypeError, match="need a contiguous device tensor"):
            call()


@pytest.mark.parametrize("missing", [True, False])
def test_without_the_extension_calls_go_through_python(missing, monkeypatch, tmp_path):
    """Not built, or built with another PyTorch: a warning, once, and the checks in Python."""
    if missing:
        monkeypatch.setattr(hb, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
    else:
        monkeypatch.setattr(torch, "__version__", "1.0.0")
    monkeypatch.setattr(hb, "_native", None)
    q = torch.zeros(2, 2, 64, dtype=torch.bfloat16)
    n = torch.zeros(2, dtype=torch.int32)
    with pytest.warns(RuntimeWarning, match="_marshal.so"), pytest.raises(TypeError, match="need a contiguous device tensor"):
        hb.hg_hydragen_attn(None, q, [], q, q, n, n, 1, q)
    with warnings.catch_warnings(), pytest.raises(TypeError, match="need a contiguous device tensor"):
        warnings.simplefilter("error")
        hb.hg_kv_append(None, q, q, q, q, n, n, 1)


@pytest.mark.gpu
@pytest.mark.parametrize("nq", [1, 3])
@pytest.mark.parametrize("cache", ["packed", "fp8", "paged"])
def test_same_results_through_either(cache, nq, monkeypatch):
    print(f"marshal: {cache} nq={nq}", flush=True)
    B, H, D, cap = 5, 2, 64, 32
    g = torch.Generator(device="cuda:0").manual_seed(5)
    r = lambda *s: torch.randn(s, generator=g, device="cuda:0").to(torch.bfloat16)      # noqa: E731
    lead = (B, H) if nq == 1 else (B, nq, H)
    Q, Kn, Vn, levels = r(*lead, D), r(*lead, D), r(*lead, D), [hb.Level(K=r(40, H, D), V=r(40, H, D), max_rows=40, max_seqs=B)]
    rows = [r(B * cap, H, D) for _ in range(2)]
    if cache == "fp8":
        rows = [x.mul(64).to(torch.float8_e4m3fn).view(torch.uint8) for x in rows]
    off = torch.arange(B, dtype=torch.int32, device="cuda:0") * cap
    table = torch.arange(B * 2, dtype=torch.int32, device="cuda:0").view(B, 2)

    def step(levels, count_known):
        ctx = hb.Context(0, hb.hg_workspace_bytes(B * nq, H, D, 8))
        if count_known:      # (else the first call sets the context's count of queries, in Python)
            ctx.set_option(hb.HG_OPT_NUM_QUERIES, nq)
            ctx._nq = nq
        K, V = (x.clone() for x in rows)
        n = torch.tensor([0, 3, 9, 20, 29], dtype=torch.int32, device="cuda:0")
        O, L = torch.zeros_like(Q), torch.zeros(lead, device="cuda:0")
        ks, scale = 1.0 / 64, 0.125
        if cache == "packed":
            hb.hg_kv_append(ctx, Kn, Vn, K, V, off, n, cap)
            hb.hg_hydragen_attn(ctx, Q, levels, K, V, off, n, cap, O, L, scale)
        elif cache == "fp8":
            hb.hg_kv_append_fp8(ctx, Kn, Vn, K, V, ks, ks, off, n, cap)
            hb.hg_hydragen_attn_fp8(ctx, Q, levels, K, V, ks, ks, off, n, cap, O, L, scale)
        else:
            kv = hb.PagedKV(K, V, table, 16)
            hb.hg_kv_append_paged(ctx, Kn, Vn, kv, n, cap)
            hb.hg_hydragen_attn_paged(ctx, Q, levels, kv, n, cap, O, L, scale)
        torch.cuda.synchronize()
        ctx.close()
        return O, L, K, V, n

    taken = []
    m = hb.native()
    names = ("attn", "attn_fp8", "attn_paged", "append", "append_fp8", "append_paged")
    watch = types.SimpleNamespace(**{f: (lambda f: lambda *a: taken.append((f, getattr(m, f)(*a))) or taken[-1][1])(f) for f in names})
    monkeypatch.setattr(hb, "_native", watch)
    first = step(levels, True)
    suffix = {"packed": "", "fp8": "_fp8", "paged": "_paged"}[cache]
    assert taken == [("append" + suffix, 0), ("attn" + suffix, 0)]
    monkeypatch.setattr(hb, "_native", hb._PythonOnly)
    second = step(levels, True)
    monkeypatch.setattr(hb, "_native", watch)
    taken.clear()
    third = step(tuple(levels), False)      # (levels in a tuple are left to Python too)
    assert taken == [("append" + suffix, 0 if nq == 1 else None), ("attn" + suffix, None)]
    for other in (second, third):
        for a, b in zip(first, other):
            assert torch.equal(a, b)
