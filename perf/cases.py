"""The calls whose speed is measured: decode-attention steps of a serving program, through the public binding.

A case is one attention call (or one KV-cache update followed by it) of one model layer.  Its fields:
  B, Hq, Hkv, D     sequences, query heads, KV heads, head dimension
  P                 rows of the block that every sequence shares (0: none)
  groups, mid       second level of a sharing tree: `groups` blocks of `mid` rows, each for its share of the sequences
  len_lo, len_hi    a sequence's own suffix rows, integers uniform on [len_lo, len_hi]
  nq                queries per sequence (1: decode; more: draft tokens verified at once)
  cache             suffix cache: "packed" or "paged" bf16 rows, "fp8" or "paged_fp8" E4M3 codes with one scale per tensor
  page              rows per page of a paged cache
  step              True: the nq new K/V rows are appended to the cache first (hg_kv_append*), as in a decode step
  fp32_out          True: O in fp32 (a caller that goes on in fp32), else bf16
Values are N(0, 1) rounded to bf16, as in this repository's workloads.
"""
import math

import torch

from paper_2402_05099_amd import binding as hb


def _case(name, B, Hq, Hkv, D, P, len_lo, len_hi, **more):
    c = dict(name=name, B=B, Hq=Hq, Hkv=Hkv, D=D, P=P, groups=0, mid=0, len_lo=len_lo, len_hi=len_hi, nq=1, cache="packed",
             page=0, step=False, fp32_out=False)
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: four sequences, one short shared prompt (launches and host work are all there is)
        _case("tiny_step", 4, 4, 4, 64, 128, 16, 16),
        # a small ragged batch with grouped heads: odd batch, prompt and suffix lengths
        _case("small_ragged_gqa", 45, 16, 2, 128, 515, 1, 150),
        # the smallest point of the paper's attention microbenchmark (Sec. 4.2: eight query heads, one KV head)
        _case("microbench_small", 256, 8, 1, 128, 1024, 128, 128),
        # a 13b-class layer serving 256 completions of one 2K prompt: the suffix rows dominate
        _case("layer_2k_prompt", 256, 40, 40, 128, 2048, 1, 256),
        # long shared document, many queries: the headline shape of bench.py
        _case("long_document", 1024, 40, 40, 128, 16384, 32, 128),
        # grouped heads at full size (64 query heads on 8 KV heads), ragged suffixes up to 512
        _case("gqa_4k_prompt", 512, 64, 8, 128, 4096, 1, 512),
        # two-level sharing tree: system prompt, 16 few-shot prompts, 128 completions each
        _case("two_level_tree", 2048, 40, 40, 128, 1024, 64, 64, groups=16, mid=512),
        # the paper's microbenchmark at its long-prefix end
        _case("microbench_large", 1024, 8, 1, 128, 16384, 128, 128),
        # a whole decode step on a paged cache (append, then attend), grouped heads, medium batch
        _case("paged_step_gqa", 128, 32, 8, 128, 2048, 1, 512, cache="paged", page=16, step=True),
        # the suffix cache kept in 8 bits, long prompt
        _case("fp8_cache_4k_prompt", 1024, 40, 40, 128, 4096, 32, 128, cache="fp8"),
        # four draft tokens per sequence verified at once
        _case("verify_4_drafts", 256, 64, 8, 128, 4096, 4, 512, nq=4),
        # head dimension 64 with fp32 results
        _case("head_dim_64", 1024, 40, 40, 64, 4096, 32, 128, fp32_out=True),
    ]


def _rows(c):
    """(suffix rows of a mean sequence that its queries see, rows per sequence the cache has room for)"""
    grown = c["nq"] if c["step"] else 0
    return 0.5 * (c["len_lo"] + c["len_hi"]) + grown, c["len_hi"] + grown


def work(c):
    kv = c["Hkv"] * c["D"]
    rows = c["B"] * c["nq"] * c["Hq"]
    mean, _ = _rows(c)
    code = 1 if c["cache"].endswith("fp8") else 2
    bytes_ = rows * c["D"] * (2 + (4 if c["fp32_out"] else 2)) + 4 * rows            # Q, O, LSE
    bytes_ += 2 * 2 * (c["P"] + c["groups"] * c["mid"]) * kv                          # shared K and V
    bytes_ += 2 * code * c["B"] * mean * kv                                           # suffix K and V
    if c["step"]:
        bytes_ += 2 * (2 + code) * c["B"] * c["nq"] * kv                              # new rows in, cache rows out
    flops = 4.0 * rows * c["D"] * (c["P"] + c["mid"] + mean)
    return {"bytes": float(bytes_), "flops": flops}


def _cost(c):
    w = work(c)
    return w["bytes"] / 5.5e12 + w["flops"] / 1.1e15


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        Hq, Hkv = rng.choice([(40, 40), (40, 40), (64, 8), (64, 8), (32, 8), (8, 1), (16, 2), (4, 4)])
        c = _case("", _log_int(rng, 4, 2048), Hq, Hkv, rng.choice([128, 128, 128, 64]), _log_int(rng, 64, 16384), 1,
                  _log_int(rng, 16, 1024))
        del c["name"]
        if rng.random() < 0.08:
            c["P"] = 0
        c["nq"] = rng.choice([1, 1, 1, 1, 2, 4])
        c["len_lo"] = max(c["nq"], rng.choice([1, c["len_hi"] // 4, c["len_hi"]]))
        if rng.random() < 0.25 and c["B"] >= 32:
            c["groups"] = rng.randint(2, 16)
            c["mid"] = _log_int(rng, 32, 1024)
        c["cache"] = rng.choice(["packed"] * 5 + ["paged"] * 2 + ["fp8"] * 2 + ["paged_fp8"])
        if c["cache"].startswith("paged"):
            c["page"] = rng.choice([16, 16, 32, 64])
        c["step"] = rng.random() < 0.3
        c["fp32_out"] = rng.random() < 0.2
        if _cost(c) <= most:
            return c


def tolerance(c):
    # O: the weights are rounded to bf16 before the product with V (2^-9 relative per term), a bf16 result once more;
    # the call against the non-decomposed one (other kernels, other order of the sums) differs by up to 2.9e-3 in the
    # 2-norm and by up to 0.015 of the root mean square in single values; stated: about four times that
    return {"rel": 1.2e-2, "max": 0.06}


class _State:
    pass


def prepare(c, seed):
    dev = "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    gc = torch.Generator()
    gc.manual_seed(int(seed))
    B, Hq, Hkv, D, nq = c["B"], c["Hq"], c["Hkv"], c["D"], c["nq"]

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.bfloat16)

    s = _State()
    s.case = c
    lead = (B, Hq) if nq == 1 else (B, nq, Hq)
    s.Q = normal(*lead, D)
    s.O = torch.empty(lead + (D,), dtype=torch.float32 if c["fp32_out"] else torch.bfloat16, device=dev)
    s.LSE = torch.empty(lead, dtype=torch.float32, device=dev)
    s.ctx = hb.Context(0, hb.hg_workspace_bytes(B * nq, Hq, D, 24))

    s.levels = []
    if c["P"]:
        s.levels.append(hb.Level(K=normal(c["P"], Hkv, D), V=normal(c["P"], Hkv, D), max_rows=c["P"], max_seqs=B))
    if c["groups"]:
        n = c["groups"]
        seq_off = [i * B // n for i in range(n + 1)]
        s.levels.append(hb.Level(
            K=normal(n * c["mid"], Hkv, D), V=normal(n * c["mid"], Hkv, D), n_blocks=n,
            kv_off=torch.tensor([i * c["mid"] for i in range(n + 1)], dtype=torch.int32).to(dev),
            seq_off=torch.tensor(seq_off, dtype=torch.int32).to(dev),
            max_rows=c["mid"], max_seqs=max(b - a for a, b in zip(seq_off, seq_off[1:]))))

    lengths = torch.randint(c["len_lo"], c["len_hi"] + 1, (B,), generator=gc, dtype=torch.int32)
    s.lengths = lengths.to(dev)
    s.max_len = int(lengths.max()) + (nq if c["step"] else 0)
    _, s.capacity = _rows(c)
    if c["step"]:
        kv_shape = (B, Hkv, D) if nq == 1 else (B, nq, Hkv, D)
        s.Knew, s.Vnew = normal(*kv_shape), normal(*kv_shape)
        s.layer_lengths = s.lengths.clone()
        room = torch.full((B,), s.capacity, dtype=torch.int32)      # every sequence has its rows reserved
    else:
        room = lengths
    s.k_scale = s.v_scale = 5.5 / 448.0 if c["cache"].endswith("fp8") else 1.0

    def cache_rows(n):
        x = normal(n, Hkv, D)
        if c["cache"].endswith("fp8"):
            x = x.mul_(448.0 / 5.5).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
        return x

    if c["cache"].startswith("paged"):
        page = c["page"]
        per_seq = (s.capacity + page - 1) // page
        table = torch.randperm(B * per_seq, generator=g, device=dev).to(torch.int32).view(B, per_seq)
        s.K, s.V = cache_rows(B * per_seq * page), cache_rows(B * per_seq * page)
        s.paged = hb.PagedKV(K=s.K, V=s.V, page_table=table, page_size=page,
                             kv_format=hb.HG_KV_E4M3 if c["cache"] == "paged_fp8" else hb.HG_KV_BF16,
                             k_scale=s.k_scale, v_scale=s.v_scale)
    else:
        offsets = torch.zeros(B, dtype=torch.int32)
        offsets[1:] = torch.cumsum(room, 0)[:-1].to(torch.int32)
        s.offsets = offsets.to(dev)
        total = int(room.sum())
        s.K, s.V = cache_rows(total), cache_rows(total)
    return s


def run(s):
    c = s.case
    lengths = s.lengths
    if c["step"]:
        # every layer appends to a cache of its own: it takes a copy of the step's lengths, which the update advances
        lengths = s.layer_lengths
        lengths.copy_(s.lengths)
        if c["cache"].startswith("paged"):
            hb.hg_kv_append_paged(s.ctx, s.Knew, s.Vnew, s.paged, lengths, s.capacity)
        elif c["cache"] == "fp8":
            hb.hg_kv_append_fp8(s.ctx, s.Knew, s.Vnew, s.K, s.V, s.k_scale, s.v_scale, s.offsets, lengths, s.capacity)
        else:
            hb.hg_kv_append(s.ctx, s.Knew, s.Vnew, s.K, s.V, s.offsets, lengths, s.capacity)
    if c["cache"].startswith("paged"):
        hb.hg_hydragen_attn_paged(s.ctx, s.Q, s.levels, s.paged, lengths, s.max_len, s.O, s.LSE)
    elif c["cache"] == "fp8":
        hb.hg_hydragen_attn_fp8(s.ctx, s.Q, s.levels, s.K, s.V, s.k_scale, s.v_scale, s.offsets, lengths, s.max_len, s.O, s.LSE)
    else:
        hb.hg_hydragen_attn(s.ctx, s.Q, s.levels, s.K, s.V, s.offsets, lengths, s.max_len, s.O, s.LSE)
    if c["step"]:
        return {"O": s.O, "LSE": s.LSE, "K": s.K, "V": s.V, "lengths": lengths}
    return {"O": s.O, "LSE": s.LSE}
