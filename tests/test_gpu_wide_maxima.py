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


def inputs(profile, seen, B, H, P, D, scale):
    """Q, K, V whose scores follow a profile for sequences with seen = 1 and hardly or not at all (2^-7, 2^-20) for others"""
    rng = np.random.default_rng(P + D)
    q, k, v = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)) for s in ((B, H, D), (P, H, D), (P, H, D)))
    q /= scale * math.sqrt(D)
    q[..., 0] = seen[:, None]
    k[..., 0] = torch.from_numpy(np.broadcast_to(PROFILES[profile](np.arange(P), P) / scale, (P,)).astype(np.float32).copy())[:, None]
    return q.bfloat16(), k.bfloat16(), v.bfloat16()


def check(q, k, v, scale, O, LSE):
    s = torch.einsum("bhd,phd->bhp", q.double(), k.double()) * scale
    lse = torch.logsumexp(s, -1)
    ref = torch.einsum("bhp,phd->bhd", torch.exp(s - lse[..., None]), v.double())
    # weights are rounded to bf16 (2^-9 relative per term) before the second product
    assert (O.cpu().double() - ref).norm() <= 2.0 ** -8 * ref.norm()
    assert (O.cpu().double() - ref).abs().max() <= 2.0 ** -7 * v.double().abs().max()
    # fp32 scores: 2^-24 relative of terms as large as the score, D of them
    assert ((LSE.cpu().double() - lse).abs() <= 1e-5 * lse.abs().clamp(min=1.0) + 1e-5).all()


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


def piece_stages(P, B, H, parts, slots, D):
    """stages of every run that a team walks without a change of column"""
    plan = hb.hg_debug_wide_plan(1, P, B, H, 1, parts, slots, D)
    runs = []
    for t in range(8 * plan["tpx"]):
        at, end, _ = hb.hg_debug_wide_team(1, P, B, H, 1, parts, slots, D, t) or (0, 0, 0)
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
