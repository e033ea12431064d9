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


@pytest.mark.parametrize("profile", PROFILES)
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("P", [31, 32, 97, 333, 1100])
@pytest.mark.parametrize("scaled_q", [False, True])      # queries that carry the scale: factor 1, by log2(e) more than 1 in the exponent
def test_moving_maxima(profile, D, P, scaled_q):
    B, H, scale = 300, 2, 1.0 if scaled_q else 1.0 / math.sqrt(D)      # two row tiles, the second one ragged
    if profile == "from_minus_inf" and P <= 70:
        pytest.skip("no finite score at all")
    rng = np.random.default_rng(P + D)
    q, k, v = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)) for s in ((B, H, D), (P, H, D), (P, H, D)))
    if scaled_q:
        q /= math.sqrt(D)
    # one column carries the profile: rows of odd sequences see a hundredth of it, so that a wavefront's rows move apart
    q[..., 0] = torch.where(torch.arange(B) % 2 == 0, 1.0, 0.0078125)[:, None]
    k[..., 0] = torch.from_numpy(np.broadcast_to(PROFILES[profile](np.arange(P), P) / scale, (P,)).astype(np.float32).copy())[:, None]
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    ctx = hb.Context(0, hb.hg_workspace_bytes(B, H, D, 16))
    ctx.set_option(hb.HG_OPT_PREFIX_KERNEL, 2)
    O, LSE = torch.empty(B, H, D, device="cuda"), torch.empty(B, H, device="cuda")
    hb.hg_prefix_attn(ctx, q.cuda(), k.cuda(), v.cuda(), O, LSE, scale=scale)
    s = torch.einsum("bhd,phd->bhp", q.double(), k.double()) * scale
    lse = torch.logsumexp(s, -1)
    ref = torch.einsum("bhp,phd->bhd", torch.exp(s - lse[..., None]), v.double())
    # weights are rounded to bf16 (2^-9 relative per term) before the second product
    assert (O.cpu().double() - ref).norm() <= 2.0 ** -8 * ref.norm()
    assert (O.cpu().double() - ref).abs().max() <= 2.0 ** -7 * v.double().abs().max()
    # fp32 scores: 2^-24 relative of terms as large as the score, D of them
    assert ((LSE.cpu().double() - lse).abs() <= 1e-5 * lse.abs().clamp(min=1.0) + 1e-5).all()
