"""fp32 kernels on the fp32 matrix instructions against the float64 oracle (1e-5 of the output's scale, the bound of the
fp32 configuration): edges of the 16-wide tiles, short and uneven reductions, head dimensions of one to eight blocks,
values of keys that nobody may see."""
import numpy as np
import pytest

from cascade_inputs import make_assignment
from oracle import cascade_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


def draw(rng, shape, std=1.0):
    return (rng.standard_normal(shape) * std).astype(np.float32)


def err(got, ref):
    got = got.cpu().numpy().astype(np.float64)
    return np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-300)


@pytest.mark.parametrize("M,N,K", [(1, 1, 4), (17, 33, 20), (16, 16, 64), (128, 192, 64), (40, 24, 132), (300, 1000, 260),
                                   (513, 520, 96)])
@pytest.mark.parametrize("epi", ["plain", "bias_gelu", "bias_residual", "swiglu"])
def test_gemm(cas, M, N, K, epi):
    import torch
    rng = np.random.default_rng(M + N + K)
    x, w = draw(rng, (M, K)), draw(rng, (N, K), K ** -0.5)
    x64 = x.astype(np.float64)
    ref = orc.linear(x64, w.astype(np.float64))
    kw, ep = {}, 0
    if epi == "swiglu":
        wu = draw(rng, (N, K), K ** -0.5)
        kw["W_up"], ep = cas.to_device(wu, "f32"), cas.EPI_SWIGLU
        ref = orc.silu(ref) * orc.linear(x64, wu.astype(np.float64))
    if "bias" in epi:
        b = draw(rng, (N,), 0.3)
        kw["bias"], ep = cas.to_device(b, "f32"), ep | cas.EPI_BIAS
        ref = ref + b
    if "gelu" in epi:
        ep |= cas.EPI_GELU_ERF
        ref = orc.gelu_erf(ref)
    if "residual" in epi:
        r = draw(rng, (M, N))
        kw["residual"], ep = cas.to_device(r, "f32"), ep | cas.EPI_RESIDUAL
        ref = ref + r
    guard = torch.full((M + 2, N), 7.0, device="cuda")
    cas.cascade_shard_gemm(None, cas.to_device(x, "f32"), cas.to_device(w, "f32"), guard[1:M + 1], epilogue=ep, **kw)
    assert err(guard[1:M + 1], ref) < TOL
    assert (guard[0] == 7.0).all() and (guard[M + 1] == 7.0).all()


def run_attention(cas, a, beta, q, k, v, B, H, Hkv, N, d, causal=True):
    import torch
    plan = cas.cascade_plan_create(B, N, beta, a, mask_kind=cas.MASK_CAUSAL if causal else cas.MASK_NONE)
    m, e = (torch.empty(B, H, beta, N, device="cuda") for _ in range(2))
    u = torch.empty(B, beta, H, N, d, device="cuda")
    o = torch.empty(B, N, H * d, device="cuda")
    cas.cascade_partial_attn(plan, q, k, v, m, e, u, H, Hkv, d, d ** -0.5)
    cas.cascade_lse_merge(plan, m, e, u, o, H, Hkv, d, row_layout=cas.ROWS_ORIGINAL)
    return m, e, u, o


@pytest.mark.parametrize("d", [4, 16, 20, 32, 48, 64, 100, 128])
@pytest.mark.parametrize("N,beta,kind", [(1, 1, "contiguous"), (15, 4, "ragged"), (67, 3, "perm"), (130, 2, "roundrobin")])
def test_attention(cas, d, N, beta, kind):
    B, H, Hkv = 2, 4, 2
    rng = np.random.default_rng(d + N)
    a = make_assignment(kind, N, beta, 4)
    q, k, v = draw(rng, (B, H, N, d)), draw(rng, (B, Hkv, N, d)), draw(rng, (B, Hkv, N, d))
    m, e, u, o = run_attention(cas, a, beta, *(cas.to_device(t, "f32") for t in (q, k, v)), B, H, Hkv, N, d)
    for b in range(B):
        for h in range(H):
            s = q[b, h].astype(np.float64) @ k[b, h // 2].astype(np.float64).T * d ** -0.5
            s[np.triu_indices(N, 1)] = -np.inf
            p = np.exp(s - s.max(1, keepdims=True))
            ref = (p / p.sum(1, keepdims=True)) @ v[b, h // 2].astype(np.float64)
            assert err(o[b, :, h * d:(h + 1) * d], ref) < TOL


def test_values_of_unseen_keys_do_not_reach_the_output(cas):
    import torch
    B, H, N, d, beta = 1, 2, 70, 32, 3
    rng = np.random.default_rng(3)
    a = make_assignment("perm", N, beta, 4)
    q, k, v = (cas.to_device(draw(rng, (B, H, N, d)), "f32") for _ in range(3))
    clean = [t.clone() for t in run_attention(cas, a, beta, q, k, v, B, H, H, N, d)]
    k[:, :, 50:], v[:, :, 50:60], v[:, :, 60:] = float("nan"), float("inf"), float("nan")
    o = run_attention(cas, a, beta, q, k, v, B, H, H, N, d)[3]
    torch.cuda.synchronize()
    assert err(o[:, :50], clean[3][:, :50].cpu().numpy().astype(np.float64)) < TOL


def fused_attention(cas, a, beta, q, k, v):
    """FUSED causal attention of q [N, H, d], k, v [N, Hkv, d] (token order): a post-norm layer whose projections select
    columns of its input (a row of the input with a NaN is all NaN: q, k and v of that token)."""
    import torch
    from cascade_inputs import CONFIGS
    N, H, d = q.shape
    Hkv = k.shape[1]
    D = (H + 2 * Hkv) * d
    cfg = CONFIGS["C1"].with_(name="select", d_model=D, n_heads=H, n_kv_heads=Hkv, head_dim=d, d_ff=16, batch=1, seq_len=N,
                              n_shards=beta, bias=False, norm="rmsnorm", norm_placement="post", index=68)
    eye = np.eye(D, dtype=np.float32)
    w = {"wq": eye[:H * d], "wk": eye[H * d:(H + Hkv) * d], "wv": eye[(H + Hkv) * d:], "wo": np.zeros((D, H * d), np.float32),
         "w_up": np.zeros((16, D), np.float32), "w_down": np.zeros((D, 16), np.float32),
         "norm1_g": np.ones(D, np.float32), "norm2_g": np.ones(D, np.float32)}
    plan, desc = cas.cascade_plan_create(1, N, beta, a), cas.make_layer_desc(cfg, cas.ATTN_FUSED)
    tensors = {n: cas.to_device(t, "f32") for n, t in w.items()}
    h_in = cas.to_device(np.concatenate([t.reshape(N, -1) for t in (q, k, v)], 1)[None], "f32")
    ws = cas.new_workspace(cas.cascade_layer_workspace_bytes(plan, desc))
    cas.cascade_layer_forward(plan, desc, cas.make_layer_weights(tensors), h_in, torch.empty_like(h_in), ws)
    o = cas.cascade_layer_attention_output(plan, desc, ws, 1, H, d).cpu().numpy()
    out = np.empty_like(o)
    out[orc.shard_plan(a, beta)[1]] = o
    return out


# one NaN token; a whole 16-key tile of them and a whole tile of 64; everything
@pytest.mark.parametrize("first,last", [(37, 38), (16, 32), (64, 128), (0, 200)])
@pytest.mark.parametrize("beta,kind", [(1, "contiguous"), (3, "perm"), (13, "contiguous")])
@pytest.mark.parametrize("d", [16, 18])                                             # matrix kernel, plain-FMA kernel
def test_nan_that_is_seen_reaches_the_output(cas, first, last, beta, kind, d):
    """Queries from the first NaN token on see it: all their outputs (and the statistics of that shard) are NaN, the
    outputs in front of it are those without it."""
    N, H, Hkv = 200, 4, 2
    rng = np.random.default_rng(last)
    a = make_assignment(kind, N, beta, 4)
    q, k, v = draw(rng, (N, H, d)), draw(rng, (N, Hkv, d)), draw(rng, (N, Hkv, d))
    clean = fused_attention(cas, a, beta, q, k, v)
    assert np.isfinite(clean).all()
    for t in (q, k, v):
        t[first:last] = np.nan
    o = fused_attention(cas, a, beta, q, k, v)
    assert np.isnan(o[first:]).all() and np.abs(o[:first] - clean[:first]).max(initial=0.0) < TOL
    heads = [np.ascontiguousarray(t.transpose(1, 0, 2)[None]) for t in (q, k, v)]
    m, e, u, o = run_attention(cas, a, beta, *(cas.to_device(t, "f32") for t in heads), 1, H, Hkv, N, d)
    assert np.isnan(o[0, first:].cpu().numpy()).all() and np.isfinite(o[0, :first].cpu().numpy()).all()
    seen = np.zeros((beta, N), bool)                                                # shard, query (packed): sees a NaN score
    perm = orc.shard_plan(a, beta)[1]
    for s in range(beta):
        bad = [t for t in np.flatnonzero(a == s) if first <= t < last]
        for r, t in enumerate(perm):
            in_shard = ((a == s) & (np.arange(N) <= t)).any()
            seen[s, r] = any(b <= t for b in bad) or (first <= t < last and in_shard)
    e, u = e[0].cpu().numpy(), u[0].cpu().numpy()                                  # [H, S, N], [S, H, N, d]
    assert np.array_equal(np.isnan(e), np.broadcast_to(seen, e.shape))
    assert np.array_equal(np.isnan(u), np.broadcast_to(seen[:, None, :, None], u.shape))


@pytest.mark.parametrize("d,scale", [(4, 0.37), (16, 0.37), (64, 0.73)])
@pytest.mark.parametrize("normalised", [False, True])
@pytest.mark.parametrize("beta", [4, 12])                                           # a query tile per workgroup, per wavefront
def test_partials_of_large_logits_fit_together(cas, d, scale, normalised, beta):
    """Integer queries and keys, so that a dot product is exact and a score is rounded by the scale alone (300 and more:
    1.5e-5 and more for half an ulp).  e and u refer to the stored m: m + log e and u / e are right to fp32 sums whatever m was
    rounded to."""
    import torch
    B, H, N = 1, 2, 150
    rng = np.random.default_rng(d)
    draw_int = lambda: rng.integers(-60 // int(d ** 0.5), 60 // int(d ** 0.5) + 1, (B, H, N, d)).astype(np.float32)
    q, k, v = draw_int(), draw_int(), draw(rng, (B, H, N, d))
    a = make_assignment("perm", N, beta, 4)
    plan = cas.cascade_plan_create(B, N, beta, a)
    m, e = (torch.empty(B, H, beta, N, device="cuda") for _ in range(2))
    u = torch.empty(B, beta, H, N, d, device="cuda")
    cas.cascade_partial_attn(plan, *(cas.to_device(t, "f32") for t in (q, k, v)), m, e, u, H, H, d, scale,
                             u_mode=cas.U_NORMALISED if normalised else cas.U_UNNORMALISED)
    m, e, u = (t.cpu().numpy().astype(np.float64) for t in (m, e, u))
    perm, scale = orc.shard_plan(a, beta)[1], float(np.float32(scale))
    largest = 0.0
    for h in range(H):
        s = (q[0, h].astype(np.float64) @ k[0, h].astype(np.float64).T * scale)[perm]
        for j in range(beta):
            keys = np.flatnonzero(a == j)
            t = np.where(keys[None, :] <= perm[:, None], s[:, keys], -np.inf)
            live = np.isfinite(t.max(1))
            ref_m = t.max(1)[live]
            p = np.exp(t[live] - ref_m[:, None])
            lse = ref_m + np.log(p.sum(1))
            largest = max(largest, np.abs(ref_m).max())
            assert np.abs(m[0, h, j][live] + np.log(e[0, h, j][live]) - lse).max() < 2e-6
            ref_u = (p / p.sum(1, keepdims=True)) @ v[0, h, keys].astype(np.float64)
            got_u = u[0, j, h][live] / (1.0 if normalised else e[0, h, j][live][:, None])
            assert np.abs(got_u - ref_u).max() < 4e-6 * np.abs(v).max()
    assert largest > 256


# a query tile per workgroup (the first), then per wavefront: shards of at most 16 rows, and of up to 64 in launches of 2048
# workgroups and more; last query tile of a workgroup short
@pytest.mark.parametrize("B,H,N,beta,d", [(1, 2, 200, 3, 20), (1, 2, 70, 5, 20), (2, 1, 33, 33, 64), (2, 4, 260, 24, 128), (3, 12, 200, 5, 32),
                                          (2, 16, 258, 4, 16)])
@pytest.mark.parametrize("causal", [False, True])
def test_partials_of_short_shards(cas, B, H, N, beta, d, causal):
    """m, e, u of every (query, shard) against float64, with and without a mask; shards of unequal sizes, some empty."""
    rng = np.random.default_rng(N + d)
    a = make_assignment("ragged", N, beta, 4)
    q, k, v = (draw(rng, (B, H, N, d)) for _ in range(3))
    m, e, u, o = run_attention(cas, a, beta, *(cas.to_device(t, "f32") for t in (q, k, v)), B, H, H, N, d, causal=causal)
    ref = [orc.partial_attention_all_pairs(*(t[b].astype(np.float64) for t in (q, k, v)), a, beta, scale=d ** -0.5,
                                           mask_kind="causal" if causal else "none") for b in range(B)]
    m_r, e_r, u_r = (np.stack([r[i] for r in ref]) for i in range(3))
    m, e = m.cpu().numpy(), e.cpu().numpy()
    dead = ~np.isfinite(m_r)
    assert (m[dead] == -np.inf).all() and (e[dead] == 0).all()
    assert np.abs(m[~dead] - m_r[~dead]).max() < TOL * np.abs(m_r[~dead]).max()
    assert np.abs(e - e_r).max() < TOL * e_r.max()
    assert err(u, e_r.transpose(0, 2, 1, 3)[..., None] * u_r) < TOL
    s = np.einsum("bhnd,bhmd->bhnm", q.astype(np.float64), k.astype(np.float64)) * d ** -0.5
    if causal:
        s[..., np.triu(np.ones((N, N), bool), 1)] = -np.inf
    p = np.exp(s - s.max(-1, keepdims=True))
    full = np.einsum("bhnm,bhmd->bnhd", p / p.sum(-1, keepdims=True), v.astype(np.float64))
    assert err(o, full.reshape(B, N, H * d)) < TOL
