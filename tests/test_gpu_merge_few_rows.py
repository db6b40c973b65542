"""Merge of few rows (a generated token's): numbers of shards around the lane groups, the pieces in flight and the 256
coefficients held at a time, empty shards, rows with nothing to merge, both forms of u; against float64."""
import numpy as np
import pytest

from launched import kernels_of

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


@pytest.mark.parametrize("S", [2, 8, 24, 300])
@pytest.mark.parametrize("norm", [False, True])
def test_weight_sum_is_rounded_once_per_shard(cas, S, norm):
    """Each shard's exp(m - n) e enters the sum w of its lane group by one fused multiply-add.  A single nonzero u makes the
    output fl(1 / w); the exponentials are read off merges of two shards; the sums are redone in extended precision."""
    import torch
    B, H, d = 3, 64, 256
    groups = 4                                                            # 256 threads, 64 lanes to a row of 256 columns
    rng = np.random.default_rng(S)
    m = -3 * rng.random((B, H, S)).astype(np.float32)
    e = (1 + 30 * rng.random((B, H, S))).astype(np.float32)
    m[:, :, 0], e[:, :, 0] = 0.0, 1.0

    def merged(m, e, u):
        n = m.shape[2]
        plan = cas.cascade_plan_create(len(m), 1, n, np.zeros(1, np.int32))
        o = torch.empty((len(m), 1, H * d), device="cuda")
        dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (m[..., None], e[..., None], u)]
        cas.cascade_lse_merge(plan, *dev, o, H, H, d, u_mode=cas.U_NORMALISED if norm else cas.U_UNNORMALISED)
        return o.view(len(m), H, d)[:, :, 7].cpu().numpy()

    # exp(m_k): maximum 0, weight 1, the second shard's u seen alone (normalised partials weigh it with e = 2^-100, which the sum loses)
    tiny = np.float32(2.0 ** -100)
    pair = np.zeros((B * S, H, 2), np.float32)
    pair[:, :, 1] = m.transpose(0, 2, 1).reshape(B * S, H)
    ones = np.zeros((B * S, H, 2), np.float32)
    ones[:, :, 0], ones[:, :, 1] = 1.0, tiny if norm else 0.0
    u = np.zeros((B * S, 2, H, 1, d), np.float32)
    u[:, 1] = 2.0 ** 100 if norm else 1.0
    c = merged(pair, ones, u).reshape(B, S, H).transpose(0, 2, 1)
    assert np.abs(c - np.exp(m.astype(np.float64))).max() < 1e-6

    u = np.zeros((B, S, H, 1, d), np.float32)
    u[:, 0] = 1.0
    total = np.zeros((B, H), np.float32)
    for g in range(groups):
        w = np.zeros((B, H), np.float32)
        for k in range(g, S, groups):
            w = (w.astype(np.longdouble) + c[:, :, k].astype(np.longdouble) * e[:, :, k]).astype(np.float32)
        total += w
    assert np.array_equal(merged(m, e, u), np.float32(1) / total)


@pytest.mark.parametrize("S,kernel", [(1, "merge_few_shards_kernel"), (16, "merge_few_shards_kernel"), (17, "merge_fewrows_kernel")])
def test_few_shards_take_the_plain_loop(cas, S, kernel):
    import torch
    plan = cas.cascade_plan_create(2, 1, S, np.zeros(1, np.int32))
    m, e, u = torch.zeros((2, 3, S, 1), device="cuda"), torch.ones((2, 3, S, 1), device="cuda"), torch.ones((2, S, 3, 1, 64), device="cuda")
    o = torch.empty((2, 1, 3 * 64), device="cuda")
    names = kernels_of(lambda: cas.cascade_lse_merge(plan, m, e, u, o, 3, 3, 64))
    assert len(names) == 1 and kernel in names[0]
