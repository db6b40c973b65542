"""bf16 shard GEMM, tiles of 128 x 96 (one and two to a CU), 192 x 128, and with SwiGLU 256 x 128 and 192 x 224; with the rotary
epilogue 128 x 96 and 256 x 96: shapes that select them on 256 CUs, ragged in rows and columns, one k-tile to many, against
the float64 oracle."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights
from oracle import cascade_oracle as orc
from test_gpu_gemm_tiles import TOL, cas, check  # noqa: F401  (fixture and the oracle comparison)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(65, 96, 64), (127, 100, 128), (128, 188, 192), (129, 964, 256), (700, 2308, 832),          # one to a CU
                                   (1500, 3076, 192), (2049, 2404, 768)])                                                 # two
@pytest.mark.parametrize("epi", ["plain", "bias_gelu", "bias_residual"])
def test_128_x_96(cas, M, N, K, epi):  # noqa: F811
    check(cas, M, N, K, epi)


@pytest.mark.parametrize("M,N,epi", [(1153, 4100, "residual"), (1344, 4096, "plain"), (5000, 772, "bias_residual"), (1200, 4228, "bias_gelu")])
def test_192_x_128(cas, M, N, epi):  # noqa: F811
    check(cas, M, N, 1600, epi)


@pytest.mark.parametrize("M,N,K", [(129, 8260, 1600), (256, 14340, 1600), (200, 9604, 2560),                   # 256 x 128
                                   (257, 14340, 1600), (333, 9604, 2048), (769 - 64, 14336, 1600)])            # 192 x 224
@pytest.mark.parametrize("epi", ["swiglu", "swiglu_residual"])
def test_swiglu(cas, M, N, K, epi):  # noqa: F811
    check(cas, M, N, K, epi)


@pytest.mark.parametrize("batch,tokens,heads,head_dim", [(1, 130, 4, 128), (1, 333, 8, 64), (4, 780, 16, 64), (3, 1000, 16, 64)])
@pytest.mark.parametrize("fused_qkv", [False, True])
def test_rotary(cas, batch, tokens, heads, head_dim, fused_qkv):  # noqa: F811
    cfg = CONFIGS["C3"].with_(name="lower", d_model=256, n_heads=heads, n_kv_heads=heads // 4, head_dim=head_dim, d_ff=512, batch=batch,
                              seq_len=tokens, n_shards=3, index=75)
    a = make_assignment("ragged", tokens, 3, 1)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a, fused_qkv=fused_qkv)
    ref = orc.layer_direct_batch(h, w, cfg)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL
