"""The persistent shared-block kernel where row maxima move: weights are taken against a maximum found in a piece's first stage, and
again where a later stage's would grow too large, by whole stages, for all rows of a wavefront or for some."""
import math

import numpy as np
import pytest
import torch

from paper_2402_05099_amd import binding as hb

pytestmark = pytest.mark.gpu

# a key's score in nats (added to noise of about 1) as a function of its row: stages hold 32 keys at D = 128, 64 at D = 64
PROFILES = {
    "rises": lambda j, P: 0.7 * j,                                        # every stage moves the maximum
    "falls": lambda j, P: -0.7 * j,
    "steps": lambda j, P: 15.0 * (j // 64),                               # one stage in two or none
    "last_key": lambda j, P: np.where(j == P - 1, 60.0, 0.0),             # the last stage, partial
    "beyond_fp32": lambda j, P: np.where(j >= P // 2, 3000.0, 0.0),       # weights against the first maximum are infinite
    "from_minus_inf": lambda j, P: np.where(j < 70, -np.inf, 0.0),        # no finite score in the first stage
}


def inputs(profile, seen, B, H, P, D, scale, Hkv=0):
    """Q, K, V whose scores follow a profile for sequences with seen = 1 and hardly or not at all (2^-7, 2^-20) for others"""
    rng = np.random.default_rng(P + D)
    q, k, v = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)) for s in ((B, H, D), (P, Hkv or H, D), (P, Hkv or H, D)))
    q /= scale * math.sqrt(D)
    q[..., 0] = seen[:, None]
    k[..., 0] = torch.from_numpy(np.broadcast_to(PROFILES[profile](np.arange(P), P) / scale, (P,)).astype(np.float32).copy())[:, None]
    return q.bfloat16(), k.bfloat16(), v.bfloat16()


def close(O, LSE, ref, lse, v_max):
    # weights are rounded to bf16 (2^-9 relative per term) before the second product
    assert (O - ref).norm() <= 2.0 ** -8 * ref.norm()
    assert (O - ref).abs().max() <= 2.0 ** -7 * v_max
    # fp32 scores: 2^-24 relative of terms as large as the score, D of them
    assert ((LSE - lse).abs() <= 1e-5 * lse.abs().clamp(min=1.0) + 1e-5).all()


def check(q, k, v, scale, O, LSE):
    s = torch.einsum("bhd,phd->bhp", q.double(), k.double()) * scale
    lse = torch.logsumexp(s, -1)
    ref = torch.einsum("bhp,phd->bhd", torch.exp(s - lse[..., None]), v.double())
    close(O.cpu().double(), LSE.cpu().double(), ref, lse, v.double().abs().max())


@pytest.mark.parametrize("profile", PROFILES)
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("P", [31, 32, 97, 333, 1100])
@pytest.mark.parametrize("scaled_q", [False, True])      # queries that carry the scale: factor 1, by log2(e) more than 1 in the exponent
def test_moving_maxima(profile, D, P, scaled_q):
    B, H, scale = 300, 2, 1.0 if scaled_q else 1.0 / math.sqrt(D)      # two row tiles, the second one ragged
    if profile == "from_minus_inf" and P <= 70:
        pytest.skip("no finite score at all")
    # rows of odd sequences see a hundredth of the profile, so that a wavefront's rows move apart
    q, k, v = inputs(profile, torch.where(torch.arange(B) % 2 == 0, 1.0, 0.0078125), B, H, P, D, scale)
    ctx = hb.Context(0, hb.hg_workspace_bytes(B, H, D, 16))
    ctx.set_option(hb.HG_OPT_PREFIX_KERNEL, 2)
    O, LSE = torch.empty(B, H, D, device="cuda"), torch.empty(B, H, device="cuda")
    hb.hg_prefix_attn(ctx, q.cuda(), k.cuda(), v.cuda(), O, LSE, scale=scale)
    check(q, k, v, scale, O, LSE)


def piece_stages(P, B, H, parts, slots, D, rows=1):
    """stages of every run that a team walks without a change of column"""
    plan = hb.hg_debug_wide_plan(1, P, B, H, rows, parts, slots, D)
    runs = []
    for t in range(8 * plan["tpx"]):
        at, end, _ = hb.hg_debug_wide_team(1, P, B, H, rows, parts, slots, D, t) or (0, 0, 0)
        while at < end:
            stop = min(end, (at // plan["n_c"] + 1) * plan["n_c"])
            runs.append(stop - at)
            at = stop
    return runs


@pytest.mark.parametrize("profile", [p for p in PROFILES if p != "falls"])
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("rows", ["even", "one_wavefront"])
@pytest.mark.parametrize("past", ["", "stage", "part", "stages_and_part"])      # what follows the last whole group of eight stages
@pytest.mark.parametrize("cut", [False, True])
def test_moving_maxima_in_long_pieces(profile, D, rows, past, cut):
    """Pieces of more than a group of eight stages: stages are taken again in unmasked steps, at every slot, after the ring has wrapped.  cut: columns
    are cut among eight teams, most of which walk the end of one column and the start of the next, from any stage; else each is one piece."""
    KT = 4096 // D                                          # 32 keys at D = 128, 64 at D = 64
    P = 24 * KT + {"": 0, "stage": KT, "part": 12, "stages_and_part": 4 * KT + 12}[past]
    B, H, scale = 300, 9, 1.0 / math.sqrt(D)
    parts, slots = (16, 2) if cut else (1, 32)
    stages = piece_stages(P, B, H, parts, slots, D)
    assert max(stages) > 17 and (len(set(stages)) >= 8) == cut
    seq = torch.arange(B)
    q, k, v = inputs(profile, torch.where(seq % 2 == 0, 1.0, 2.0 ** -7) if rows == "even" else torch.where((seq >= 64) & (seq < 96), 1.0, 2.0 ** -20),
                     B, H, P, D, scale)
    ctx = hb.Context(0, hb.hg_workspace_bytes(B, H, D, parts))
    ctx.set_option(hb.HG_OPT_PREFIX_KERNEL, 2)
    ctx.set_option(hb.HG_OPT_WIDE_SLOTS, slots)
    O, LSE = torch.empty(B, H, D, device="cuda"), torch.empty(B, H, device="cuda")
    hb.hg_prefix_attn(ctx, q.cuda(), k.cuda(), v.cuda(), O, LSE, scale=scale)
    check(q, k, v, scale, O, LSE)


# name: (sequences, queries per sequence, query heads, KV heads), 300 or 400 query rows per KV head
ROLES = {"vector": (300, 1, 9, 9), "tiles_16": (100, 1, 36, 9), "tiles_32": (20, 5, 36, 9)}


@pytest.mark.parametrize("profile", ["rises", "steps", "last_key"])
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("role", ROLES)
def test_moving_maxima_beside_a_suffix(profile, D, role):
    """The same in the launch that shared block and suffix have in common, which compiles the shared block's source once more per kind of suffix role."""
    B, nq, H, Hkv = ROLES[role]
    KT = 4096 // D
    P, G, scale, lo, hi = 24 * KT + 12, H // Hkv, 1.0 / math.sqrt(D), 24, 40
    options = {hb.HG_OPT_FUSED_KERNEL: 1, hb.HG_OPT_WIDE_SLOTS: 2}
    room = hb.hg_workspace_bytes(B * nq, H, D, 16)
    plan = hb.hg_debug_fused_plan([(1, P, B)], B, nq, H, Hkv, D, hi, workspace_bytes=room, options=options)
    assert plan["way"] == "combined" and plan["mfma"] == (role != "vector")
    assert max(piece_stages(P, B, Hkv, 16, 2, D, nq * G)) > 17
    seen = torch.where(torch.arange(B * nq) % 2 == 0, 1.0, 0.0078125)
    q, k, v = inputs(profile, seen, B * nq, H, P, D, scale, Hkv)
    g = torch.Generator().manual_seed(D)
    lengths = torch.randint(lo, hi + 1, (B,), generator=g, dtype=torch.int32)
    ks, vs = (torch.randn(B, hi, Hkv, D, generator=g).bfloat16() for _ in range(2))     # room for hi rows each
    ctx = hb.Context(0, room)
    for o, value in options.items():
        ctx.set_option(o, value)
    lead = (B, H) if nq == 1 else (B, nq, H)
    O, LSE = torch.empty(*lead, D, device="cuda"), torch.empty(*lead, device="cuda")
    level = hb.Level(K=k.cuda(), V=v.cuda(), max_rows=P, max_seqs=B)
    hb.hg_hydragen_attn(ctx, q.view(*lead, D).cuda(), [level], ks.view(-1, Hkv, D).cuda(), vs.view(-1, Hkv, D).cuda(),
                        (torch.arange(B, dtype=torch.int32) * hi).cuda(), lengths.cuda(), hi, O, LSE, scale)
    q = q.double().view(B, nq, Hkv, G, D)
    s = torch.cat([torch.einsum("bthgd,phd->bthgp", q, k.double()), torch.einsum("bthgd,bjhd->bthgj", q, ks.double())], -1) * scale
    # query t of nq is suffix token length - nq + t and sees no later one
    sees = lengths[:, None] - (nq - 1 - torch.arange(nq))
    s[..., P:].masked_fill_((torch.arange(hi) >= sees[..., None])[:, :, None, None], -math.inf)
    lse = torch.logsumexp(s, -1)
    w = torch.exp(s - lse[..., None])
    ref = torch.einsum("bthgp,phd->bthgd", w[..., :P], v.double()) + torch.einsum("bthgj,bjhd->bthgd", w[..., P:], vs.double())
    close(O.cpu().double().view(ref.shape), LSE.cpu().double().view(lse.shape), ref, lse, max(v.abs().max().item(), vs.abs().max().item()))
