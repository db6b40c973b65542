"""bf16 shard GEMM of few rows (the reduction split over the wavefronts of a workgroup) against the float64 oracle:
edges of its 16-row and 16-column blocks, short and uneven reductions, every epilogue, row maps, weight segments."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, round_to_bf16
from oracle import cascade_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 results: a handful of 2^-9 roundings on the output's scale


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


def draw(rng, shape, std=1.0):
    return round_to_bf16((rng.standard_normal(shape) * std).astype(np.float32))


def close(got, ref):
    got = got.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() / np.abs(ref).max() < TOL


# K / 64 below, at and above the 8 wavefronts and their ring of pieces; N ragged in its last block; two column blocks
# per workgroup from 6144 columns.  One round of workgroups for the plain epilogues but (8 and 20, 24580, 2048) and
# (32, 24587, 64), which the tile kernels take; SwiGLU launches of more than 4096 columns are of several rounds and theirs
@pytest.mark.parametrize("M,N,K", [(1, 1003, 64), (15, 48, 448), (16, 52, 512), (17, 1000, 576), (32, 20, 2752), (33, 1, 768),
                                   (64, 1001, 3072), (5, 6150, 192), (31, 6147, 128), (64, 6160, 640), (8, 24580, 2048),
                                   (20, 24580, 2048), (32, 24587, 64), (63, 8208, 2112)])
@pytest.mark.parametrize("epi", ["plain", "bias_gelu", "bias_residual", "swiglu", "swiglu_residual"])
def test_blocks_and_epilogues(cas, M, N, K, epi):
    import torch
    rng = np.random.default_rng(M * 7 + N + K)
    x, w = draw(rng, (M, K)), draw(rng, (N, K), K ** -0.5)
    x64, ref = x.astype(np.float64), None
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
    close(guard[1:M + 1], ref)
    assert (guard[0] == 7.0).all() and (guard[M + 1] == 7.0).all()


@pytest.mark.parametrize("B,N", [(1, 37), (3, 21), (2, 32)])
def test_row_maps(cas, B, N):
    """Gather on the read, residual and store in the caller's order, several sequences in one block of rows."""
    import torch
    K, F, beta = 320, 200, 4
    rng = np.random.default_rng(N)
    a = make_assignment("ragged", N, beta, 3)
    plan = cas.cascade_plan_create(B, N, beta, a)
    _, perm, _ = orc.shard_plan(a, beta)
    rows = np.concatenate([b * N + perm for b in range(B)])
    x, w, r = draw(rng, (B * N, K)), draw(rng, (F, K), 0.06), draw(rng, (B * N, F))
    X, W, R = (cas.to_device(t, "bf16") for t in (x, w, r))
    y = orc.linear(x.astype(np.float64), w.astype(np.float64))
    Y = torch.empty(B * N, F, dtype=torch.bfloat16, device="cuda")
    cas.cascade_shard_gemm(plan, X, W, Y, x_rows=cas.ROWS_ORIGINAL)
    close(Y, y[rows])
    cas.cascade_shard_gemm(plan, X, W, Y, x_rows=cas.ROWS_ORIGINAL, y_rows=cas.ROWS_ORIGINAL, res_rows=cas.ROWS_ORIGINAL,
                           residual=R, epilogue=cas.EPI_RESIDUAL)
    close(Y, y + r.astype(np.float64))
    Y.copy_(R)                                                                      # in place on the residual
    cas.cascade_shard_gemm(plan, X, W, Y, residual=Y, epilogue=cas.EPI_RESIDUAL)
    close(Y, y + r.astype(np.float64))


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("fused_qkv", [False, True])
@pytest.mark.parametrize("tokens,bias", [(1, False), (23, True), (64, False)])
def test_layer_of_a_short_prompt(cas, head_dim, fused_qkv, tokens, bias):
    """Rotary epilogue with the q, k, v weights apart and as one matrix; every projection of the layer takes few rows."""
    cfg = CONFIGS["C3"].with_(name="short", d_model=256, n_heads=4, n_kv_heads=2, head_dim=head_dim, d_ff=512, bias=bias,
                              seq_len=tokens, n_shards=min(3, tokens), index=61)
    from cascade_inputs import make_hidden, make_layer_weights
    a = make_assignment("ragged", tokens, cfg.n_shards, 1)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a, fused_qkv=fused_qkv)
    ref = orc.layer_sharded_batch(h, w, cfg, a, cfg.n_shards)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL


# two rounds of workgroups and more, which need a longer reduction; each of the block counts with 16, 32 and 64 rows
@pytest.mark.parametrize("M,N,K", [(16, 10250, 2112), (3, 20011, 2048), (33, 6100, 832), (64, 8190, 2112), (30, 8190, 192)])
@pytest.mark.parametrize("epi", ["plain", "bias_residual"])
def test_more_rounds(cas, M, N, K, epi):
    test_blocks_and_epilogues(cas, M, N, K, epi)


@pytest.mark.parametrize("M,N,K", [(16, 5003, 2112), (3, 20011, 2048), (63, 4090, 2112), (31, 4090, 192), (8, 8210, 8192)])
@pytest.mark.parametrize("epi", ["swiglu", "swiglu_residual"])
def test_more_rounds_of_pairs(cas, M, N, K, epi):
    test_blocks_and_epilogues(cas, M, N, K, epi)
