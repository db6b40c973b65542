"""bf16 shard GEMM, tile choice: the 128 x 128 tiles (one workgroup per CU with three k-tiles in flight, or two per CU)
and the wide tiles at reductions long enough to select them, against the float64 oracle."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights, round_to_bf16
from oracle import cascade_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 results: a handful of 2^-9 roundings on the output's scale


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


def draw(rng, shape, std=1.0):
    return round_to_bf16((rng.standard_normal(shape, dtype=np.float32) * np.float32(std)))


def check(cas, M, N, K, epi):
    import torch
    rng = np.random.default_rng(M + 3 * N + K)
    x, w = draw(rng, (M, K)), draw(rng, (N, K), K ** -0.5)
    x64 = x.astype(np.float64)
    ref = orc.linear(x64, w.astype(np.float64))
    kw, ep = {}, 0
    if "swiglu" in epi:
        wu = draw(rng, (N, K), K ** -0.5)
        kw["W_up"], ep = cas.to_device(wu, "bf16"), cas.EPI_SWIGLU
        ref = orc.silu(ref) * orc.linear(x64, wu.astype(np.float64))
    if "bias" in epi:
        b = draw(rng, (N,), 0.3)
        kw["bias"], ep = cas.to_device(b, "bf16"), ep | cas.EPI_BIAS
        ref = ref + b.astype(np.float64)
    if "gelu" in epi:
        ep |= cas.EPI_GELU_ERF
        ref = orc.gelu_erf(ref)
    if "residual" in epi:
        r = draw(rng, (M, N))
        kw["residual"], ep = cas.to_device(r, "bf16"), ep | cas.EPI_RESIDUAL
        ref = ref + r.astype(np.float64)
    guard = torch.full((M + 2, N), 7.0, dtype=torch.bfloat16, device="cuda")       # rows around Y stay untouched
    cas.cascade_shard_gemm(None, cas.to_device(x, "bf16"), cas.to_device(w, "bf16"), guard[1:M + 1], epilogue=ep, **kw)
    got = guard[1:M + 1].float().cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() / np.abs(ref).max() < TOL
    assert (guard[0] == 7.0).all() and (guard[M + 1] == 7.0).all()


# one to five k-tiles (the pipeline is three deep), tile edges in rows and columns, one and two workgroups per CU
@pytest.mark.parametrize("M,N,K", [(65, 128, 64), (127, 132, 128), (128, 1000, 192), (129, 260, 256), (255, 124, 320),
                                   (600, 2052, 832), (1300, 3404, 64), (1025, 3972, 192), (2049, 2052, 576), (1000, 2308, 192)])
@pytest.mark.parametrize("epi", ["plain", "bias_gelu", "bias_residual", "swiglu", "swiglu_residual"])
def test_small_tiles(cas, M, N, K, epi):
    check(cas, M, N, K, epi)


# 256 x 128 and wider tiles: more than 512 tiles of 128 x 128 and a reduction above 1536
@pytest.mark.parametrize("M,N,epi", [(700, 9600, "swiglu"), (1000, 13728, "bias_gelu"), (1000, 12352, "residual"),
                                     (1300, 10804, "bias_gelu"), (2000, 12352, "bias_residual"), (1700, 14416, "plain"),
                                     (2700, 5000, "residual"), (2700, 9600, "swiglu_residual"), (4500, 2100, "bias_gelu")])
def test_wide_tiles(cas, M, N, epi):
    check(cas, M, N, 1600, epi)


@pytest.mark.parametrize("batch,tokens,d_model,heads,head_dim", [(1, 300, 256, 4, 64), (1, 130, 512, 4, 128), (3, 700, 1024, 16, 64)])
@pytest.mark.parametrize("fused_qkv", [False, True])
def test_rotary_epilogue_of_the_small_tiles(cas, batch, tokens, d_model, heads, head_dim, fused_qkv):
    cfg = CONFIGS["C3"].with_(name="tiles", d_model=d_model, n_heads=heads, n_kv_heads=heads // 4, head_dim=head_dim, d_ff=512,
                              batch=batch, seq_len=tokens, n_shards=3, index=62)
    a = make_assignment("ragged", tokens, 3, 1)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a, fused_qkv=fused_qkv)
    ref = orc.layer_direct_batch(h, w, cfg)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL
