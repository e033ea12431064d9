"""The vector-ALU suffix kernel where row maxima move from batch to batch: sums over 8-bit rows are rescaled only when a score passes the
maximum by 2^8; the lanes that hold parts of a row are combined by swaps of registers."""
import math

import pytest
import torch

from paper_2402_05099_amd import binding as hb

pytestmark = pytest.mark.gpu

PROFILES = {"flat": 0.0, "rises": 0.5, "rises_steeply": 9.0, "falls": -0.5, "falls_steeply": -9.0}      # nats per key


@pytest.mark.parametrize("profile", PROFILES)
@pytest.mark.parametrize("codes", [False, True])
@pytest.mark.parametrize("D, Hq, Hkv", [(128, 3, 3), (64, 3, 3), (128, 4, 2), (128, 8, 2)])      # 1, 2 and 4 query heads of a KV head per work item
def test_moving_maxima(profile, codes, D, Hq, Hkv):
    torch.manual_seed(D + Hq)
    lens = torch.tensor([1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 48, 49, 64, 65, 100, 255, 256, 257, 300], dtype=torch.int32)
    offs = torch.cumsum(lens, 0).to(torch.int32) - lens
    B, T = len(lens), int(lens.sum())
    k_scale, v_scale = 16.0, 0.01
    q, k, v = torch.randn(B, Hq, D), torch.randn(T, Hkv, D), torch.randn(T, Hkv, D)
    # one column carries the profile, at a hundredth in odd sequences
    q[..., 0] = torch.where(torch.arange(B) % 2 == 0, 1.0, 0.0078125)[:, None]
    pos = torch.cat([torch.arange(int(n)) for n in lens])
    k[..., 0] = (PROFILES[profile] * (pos - pos.float().mean()) * math.sqrt(D))[:, None]
    q = q.bfloat16()
    ctx = hb.Context(0, hb.hg_workspace_bytes(B, Hq, D, 4))
    ctx.set_option(hb.HG_OPT_SUFFIX_KERNEL, 1)
    O, LSE = torch.empty(B, Hq, D, device="cuda"), torch.empty(B, Hq, device="cuda")
    if codes:
        k8 = (k / k_scale).clamp(-448, 448).to(torch.float8_e4m3fn)
        v8 = (v / v_scale).clamp(-448, 448).to(torch.float8_e4m3fn)
        hb.hg_suffix_attn_fp8(ctx, q.cuda(), k8.view(torch.uint8).cuda(), v8.view(torch.uint8).cuda(), k_scale, v_scale, offs.cuda(), lens.cuda(),
                              int(lens.max()), O, LSE)
        k, v = k8.double() * k_scale, v8.double() * torch.tensor(v_scale).double()
    else:
        k, v = k.bfloat16(), v.bfloat16()
        hb.hg_suffix_attn(ctx, q.cuda(), k.cuda(), v.cuda(), offs.cuda(), lens.cuda(), int(lens.max()), O, LSE)
        k, v = k.double(), v.double()
    O, LSE = O.cpu().double(), LSE.cpu().double()
    G = Hq // Hkv
    for b in range(B):
        a, e = int(offs[b]), int(offs[b] + lens[b])
        s = torch.einsum("hd,nhd->hn", q[b].double(), k[a:e].repeat_interleave(G, 1)) / math.sqrt(D)
        lse = torch.logsumexp(s, -1)
        ref = torch.einsum("hn,nhd->hd", torch.exp(s - lse[:, None]), v[a:e].repeat_interleave(G, 1))
        # fp32 scores: D roundings of 2^-24 relative to partial sums up to sum |q| |k| / sqrt(D), sqrt(D) of them in the end; bf16 rows: weights rounded
        # to bf16 (2^-9 relative per term)
        size = (q[b].double().abs() @ k[a:e].abs().repeat_interleave(G, 1).amax(0).T).diagonal().amax() / math.sqrt(D)
        err = 2.0 ** -20 * float(size) + 1e-6
        assert ((LSE[b] - lse).abs() <= err).all(), (b, (LSE[b] - lse).abs().max(), err)
        bound = (2 * err + (0.0 if codes else 2.0 ** -8)) * v[a:e].abs().amax()
        assert ((O[b] - ref).abs() <= bound).all(), (b, (O[b] - ref).abs().max(), bound)
