"""bf16 shard GEMM, tiles of 128 x 96 (one and two to a CU), 192 x 128, and with SwiGLU 256 x 128 and 192 x 224; with the rotary
epilogue 128 x 96 and 256 x 96: each shape's tile by name on 256 CUs, ragged in rows and columns, one k-tile to many, against
the float64 oracle."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights
from launched import gemm_tiles, kernels_of, layer_kernels
from oracle import cascade_oracle as orc
from test_gpu_gemm_tiles import TOL, cas, check  # noqa: F401  (fixture and the oracle comparison)

pytestmark = pytest.mark.gpu


def tile_of(cas, M, N, K, epi):  # noqa: F811
    """Rows and columns of the tile that the GEMM runs in."""
    import torch
    t = lambda *shape: torch.zeros(shape, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    kw, ep = {}, 0
    if "swiglu" in epi:
        kw["W_up"], ep = t(N, K), cas.EPI_SWIGLU
    if "bias" in epi:
        kw["bias"], ep = t(N), ep | cas.EPI_BIAS
    if "gelu" in epi:
        ep |= cas.EPI_GELU_ERF
    if "residual" in epi:
        kw["residual"], ep = t(M, N), ep | cas.EPI_RESIDUAL
    x, w, y = t(M, K), t(N, K), t(M, N)
    (tile,) = gemm_tiles(kernels_of(lambda: cas.cascade_shard_gemm(None, x, w, y, epilogue=ep, **kw)))
    return tile


@pytest.mark.parametrize("M,N,K", [(65, 96, 64), (127, 100, 128), (128, 188, 192), (129, 964, 256), (700, 2308, 832),          # one to a CU
                                   (1500, 3076, 192), (2049, 2404, 768)])                                                 # two
@pytest.mark.parametrize("epi", ["plain", "bias_gelu", "bias_residual"])
def test_128_x_96(cas, M, N, K, epi):  # noqa: F811
    assert tile_of(cas, M, N, K, epi) == (128, 96)
    check(cas, M, N, K, epi)


@pytest.mark.parametrize("M,N,epi", [(1220, 4228, "bias_residual"), (1500, 4004, "residual"), (1280, 4100, "plain"), (1153, 4228, "bias_gelu")])
def test_192_x_128(cas, M, N, epi):  # noqa: F811
    assert tile_of(cas, M, N, 1600, epi) == (192, 128)
    check(cas, M, N, 1600, epi)


@pytest.mark.parametrize("M,N,K,epi", [(1040, 4096, 4096, "plain"), (1344, 4096, 4096, "bias_residual"), (900, 6144, 4096, "bias"),
                                       (1152, 4096, 2048, "residual")])
def test_a_short_last_row_of_wide_tiles_keeps_them(cas, M, N, K, epi):  # noqa: F811
    assert tile_of(cas, M, N, K, epi) != (192, 128)


@pytest.mark.parametrize("M,N,K,tile", [(129, 10500, 1600, (256, 128)), (200, 10500, 2560, (256, 128)), (256, 14340, 1600, (256, 128)),
                                        (257, 9604, 2048, (192, 224)), (333, 9604, 2048, (192, 224)), (705, 14336, 1600, (192, 224))])
@pytest.mark.parametrize("epi", ["swiglu", "swiglu_residual"])
def test_swiglu(cas, M, N, K, tile, epi):  # noqa: F811
    assert tile_of(cas, M, N, K, epi) == tile
    check(cas, M, N, K, epi)


@pytest.mark.parametrize("batch,tokens,heads,head_dim,tile", [(1, 130, 4, 128, (128, 96)), (1, 333, 8, 64, (128, 96)),
                                                              (4, 780, 16, 64, (256, 96)), (3, 1000, 16, 64, (256, 96))])
@pytest.mark.parametrize("fused_qkv", [False, True])
def test_rotary(cas, batch, tokens, heads, head_dim, tile, fused_qkv):  # noqa: F811
    cfg = CONFIGS["C3"].with_(name="lower", d_model=256, n_heads=heads, n_kv_heads=heads // 4, head_dim=head_dim, d_ff=512, batch=batch,
                              seq_len=tokens, n_shards=3, index=75)
    a = make_assignment("ragged", tokens, 3, 1)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a, fused_qkv=fused_qkv)
    ref = orc.layer_direct_batch(h, w, cfg)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL
    assert gemm_tiles(layer_kernels(cas, cfg, w, h, a, fused_qkv=fused_qkv))[0] == tile
