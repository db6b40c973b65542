"""bf16 shard GEMM, epilogues that store from the accumulators: rows scattered and residual rows gathered through the plan's map
where a tile holds several sequences, outputs and residuals that start on 8-byte boundaries only, odd numbers of column
blocks per wavefront, last columns inside a lane's eight; several tiles per workgroup; the wide tiles by name.  Against the float64
oracle."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights, round_to_bf16
from launched import gemm_tiles, kernels_of, layer_kernels
from oracle import cascade_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 results: a handful of 2^-9 roundings on the output's scale


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


def draw(rng, shape, std=1.0):
    return round_to_bf16(rng.standard_normal(shape, dtype=np.float32) * np.float32(std))


def compare(cas, batch, N, K, epi, offset):
    """Sequences of 100 rows against float64; the tile the GEMM ran in."""
    import torch
    n = 100
    M = batch * n
    rng = np.random.default_rng(N + batch)
    plan = cas.cascade_plan_create(batch, n, 5, make_assignment("ragged", n, 5, 3))
    perm = np.argsort(make_assignment("ragged", n, 5, 3), kind="stable")
    rows = (np.arange(batch)[:, None] * n + perm).ravel()                      # original row of every packed one
    x, w = draw(rng, (M, K)), draw(rng, (N, K), K ** -0.5)
    wu = draw(rng, (N, K), K ** -0.5) if "swiglu" in epi else None
    b, r = draw(rng, (N,), 0.3), draw(rng, (M, N))
    check = np.unique(np.concatenate([np.arange(0, M, 37), np.arange(M - 3, M)]))   # packed rows compared in float64
    ref = orc.linear(x[check].astype(np.float64), w.astype(np.float64))
    ep = 0
    if wu is not None:
        ep, ref = cas.EPI_SWIGLU, orc.silu(ref) * orc.linear(x[check].astype(np.float64), wu.astype(np.float64))
    if "bias" in epi:
        ep, ref = ep | cas.EPI_BIAS, ref + b.astype(np.float64)
    if "gelu" in epi:
        ep, ref = ep | cas.EPI_GELU_ERF, orc.gelu_erf(ref)
    if "residual" in epi:
        ep, ref = ep | cas.EPI_RESIDUAL, ref + r[rows[check]].astype(np.float64)
    out = torch.full((M * N + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    res = torch.empty(M * N + 16, dtype=torch.bfloat16, device="cuda")
    y = out[8 + offset:8 + offset + M * N].view(M, N)
    res = res[8 + offset:8 + offset + M * N].view(M, N)
    res.copy_(cas.to_device(r, "bf16"))
    X, W, WU, b = (None if t is None else cas.to_device(t, "bf16") for t in (x, w, wu, b if "bias" in epi else None))
    call = lambda: cas.cascade_shard_gemm(plan, X, W, y, W_up=WU, bias=b, residual=res if "residual" in epi else None, epilogue=ep,  # noqa: E731
                                          y_rows=cas.ROWS_ORIGINAL, res_rows=cas.ROWS_ORIGINAL)
    tiles = gemm_tiles(kernels_of(call))
    got = y.float().cpu().numpy()[rows[check]]
    assert np.abs(got - ref).max() / np.abs(ref).max() < TOL
    assert (out[:8 + offset] == 7.0).all() and (out[8 + offset + M * N:] == 7.0).all()
    return tiles


# 128 x 96 (three column blocks per wavefront), 128 x 128 with one and two workgroups per CU, 192 and 224 columns
@pytest.mark.parametrize("batch,N,K", [(3, 192, 128), (3, 132, 192), (3, 200, 64), (41, 768, 768), (45, 2308, 768), (21, 6152, 2048),
                                       (41, 4104, 2048)])
@pytest.mark.parametrize("epi", ["plain", "residual", "bias_gelu", "bias_residual"])
@pytest.mark.parametrize("offset", [0, 4])
def test_rows_and_alignment(cas, batch, N, K, epi, offset):
    compare(cas, batch, N, K, epi, offset)


# the wide tiles and those of SwiGLU by name; last columns inside a lane's eight and whole ones
@pytest.mark.parametrize("batch,N,K,tile,epis", [(14, 4100, 2048, (256, 128), "plain residual bias_gelu bias_residual"),
                                                 (20, 4096, 2048, (256, 128), "plain residual bias_gelu bias_residual"),
                                                 (41, 4104, 2048, (256, 192), "plain bias_gelu bias_residual"), (20, 6148, 1600, (256, 224), "plain bias_residual"),
                                                 (81, 4092, 2048, (256, 256), "plain bias_residual"),
                                                 (2, 10500, 2560, (256, 128), "swiglu swiglu_residual"), (11, 4100, 2048, (192, 224), "swiglu swiglu_residual"),
                                                 (14, 4100, 2048, (256, 224), "swiglu swiglu_residual"), (20, 4096, 2048, (256, 256), "swiglu swiglu_residual"),
                                                 (3, 132, 192, (128, 128), "swiglu swiglu_residual")])
@pytest.mark.parametrize("offset", [0, 4])
def test_wide_tiles_and_swiglu(cas, batch, N, K, tile, epis, offset):
    for epi in epis.split():
        assert compare(cas, batch, N, K, epi, offset) == [tile], epi


# rotary embedding in the epilogue with biases: q, k rotated behind theirs, v with its own
@pytest.mark.parametrize("batch,tokens,heads,head_dim,tile", [(1, 130, 4, 128, (128, 96)), (4, 780, 16, 64, (256, 96)), (3, 1000, 16, 64, (256, 96))])
@pytest.mark.parametrize("fused_qkv", [False, True])
def test_rotary_with_biases(cas, batch, tokens, heads, head_dim, tile, fused_qkv):
    cfg = CONFIGS["C3"].with_(name="biases", d_model=256, n_heads=heads, n_kv_heads=heads // 4, head_dim=head_dim, d_ff=512, bias=True, act="gelu",
                              norm="layernorm", batch=batch, seq_len=tokens, n_shards=3, index=76)
    a = make_assignment("ragged", tokens, 3, 1)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a, fused_qkv=fused_qkv)
    ref = orc.layer_direct_batch(h, w, cfg)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL
    assert gemm_tiles(layer_kernels(cas, cfg, w, h, a, fused_qkv=fused_qkv))[0] == tile
