"""Merge of few rows (a generated token's): numbers of shards around the lane groups, the pieces in flight and the 256
coefficients held at a time, empty shards, rows with nothing to merge, both forms of u; against float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


@pytest.mark.parametrize("d", [16, 64, 128, 256])
@pytest.mark.parametrize("S", [1, 3, 8, 63, 65, 256, 257, 600])
@pytest.mark.parametrize("norm", [False, True])
def test_merge(cas, S, d, norm):
    import torch
    B, H = 2, 5
    g = torch.Generator(device="cuda").manual_seed(S * d)
    m = 3 * torch.randn((B, H, S, 1), device="cuda", generator=g)
    e = 1 + 30 * torch.rand((B, H, S, 1), device="cuda", generator=g)
    u = torch.randn((B, S, H, 1, d), device="cuda", generator=g)
    dead = torch.rand((B, H, S, 1), device="cuda", generator=g) < 0.3
    dead[1, 2] = True                                                     # a row without any key
    m.masked_fill_(dead, -float("inf"))
    e.masked_fill_(dead, 0.0)
    u.masked_fill_(dead[..., None].transpose(1, 2), 0.0)
    plan = cas.cascade_plan_create(B, 1, S, np.zeros(1, np.int32))
    o = torch.full((B, 1, H * d), 7.0, device="cuda")
    cas.cascade_lse_merge(plan, m, e, u, o, H, H, d, u_mode=cas.U_NORMALISED if norm else cas.U_UNNORMALISED)
    c = torch.exp(m.double() - m.double().amax(2, keepdim=True).clamp_min(-1e300))
    w = (c * e.double()).sum(2)                                           # [B, H, 1]
    cu = c * e.double() if norm else c
    ref = torch.einsum("bhs,bshd->bhd", cu[..., 0], u[:, :, :, 0].double()) / w.clamp_min(1e-300)
    err = (o.view(B, H, d).double() - ref).abs().max() / ref.abs().max()
    assert err < 1e-5                                                     # fp32 sums of up to 600 terms
    assert (o.view(B, H, d)[1, 2] == 0).all()
