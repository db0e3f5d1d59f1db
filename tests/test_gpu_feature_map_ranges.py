"""The feature map's split of tokens over workgroups: ranges of one, two and many tiles, ragged ends, head groups that are not full."""
import pytest
import torch

import paper_2605_16579_amd as A

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,L,D", [
    (1, 1, 1, 128), (1, 3, 33, 128), (2, 5, 31, 64),           # one tile per workgroup, last head group half empty
    (1, 12, 4680, 128), (1, 9, 6000, 64),                      # two tiles, the last range shorter
    (8, 5, 3001, 128), (8, 12, 4680, 128), (8, 24, 3120, 128),     # many; as many workgroups as slots, one round all the same
    (16, 24, 1560, 128), (43, 3, 777, 64), (264, 3, 70, 128)])     # rounds of short ranges; more workgroups than slots with one range each
@pytest.mark.parametrize("rope", [True, False])
def test_feature_map(B, H, L, D, rope):
    g = torch.Generator(device="cuda")
    g.manual_seed(L + H)
    x = torch.randn((B, L, H, D), generator=g, device="cuda").to(torch.bfloat16)
    W = (torch.randn((H, D, D), generator=g, device="cuda") / D ** 0.5).to(torch.bfloat16)
    angle = torch.rand((L, D // 2), generator=g, device="cuda") * 6.28
    cs, sn = (angle.cos(), angle.sin()) if rope else (None, None)
    y = torch.full_like(x, float("nan"))
    A.arl2_feature_map(x, W, cs, sn, y)
    worst = 0.0
    for h in range(H):                                         # plain fp32, head by head
        ref = x[:, :, h].float() @ W[h].float().T
        if rope:
            even, odd = ref[..., 0::2].clone(), ref[..., 1::2].clone()
            ref[..., 0::2], ref[..., 1::2] = even * cs - odd * sn, even * sn + odd * cs
        worst = max(worst, float((y[:, :, h].float() - ref).abs().max() / ref.abs().max()))
    assert worst <= 2 ** -8, f"{worst:.2e}"                    # one rounding to bf16, 2^-9 of the value
