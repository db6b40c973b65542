"""Shard GEMM of few rows with the rotary epilogue (angles computed in the GEMM): row blocks of 16 and the 64-row limit,
several sequences, large positions, bias, columns behind the rotated ones, head dimensions it takes (32 .. 256) and the ones
that stay with the pass behind the GEMM (48, a last head cut short).  Every bf16 route's angles at positions up to 2^24.
Against the float64 oracle."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_hidden, make_layer_weights
from launched import kernels_of
from oracle import cascade_oracle as orc
from test_gpu_few_rows import cas, close, draw  # noqa: F401  (fixture and helpers)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N", [(1, 1), (4, 1), (15, 1), (1, 17), (3, 11), (64, 1), (13, 5)])
@pytest.mark.parametrize("H,rot,d,tail,K,bias", [(48, 40, 128, 0, 2048, False), (3, 2, 32, 0, 64, True), (5, 5, 64, 0, 832, True),
                                                (3, 2, 256, 0, 512, False), (4, 3, 48, 0, 128, True), (4, 3, 32, 16, 128, False)])
def test_rotated_rows(cas, B, N, H, rot, d, tail, K, bias):  # noqa: F811
    import torch
    rng = np.random.default_rng(B * 100 + N + H * d)
    M, cols = B * N, H * d + tail
    pos = rng.integers(0, 1 << 20, N).astype(np.int32)
    plan = cas.cascade_plan_create(B, N, 1, np.zeros(N, np.int32), positions=pos)
    x, w, b = draw(rng, (M, K)), draw(rng, (cols, K), K ** -0.5), draw(rng, (cols,), 0.3)
    y = orc.linear(x.astype(np.float64), w.astype(np.float64)) + (b.astype(np.float64) if bias else 0.0)
    ref = y.copy()
    for h in range(rot):
        ref[:, h * d:(h + 1) * d] = orc.rope(y[:, h * d:(h + 1) * d], np.tile(pos, B), 500000.0)
    guard = torch.full((M + 2, cols), 7.0, dtype=torch.bfloat16, device="cuda")    # rows around Y stay untouched
    kw = {"bias": cas.to_device(b, "bf16")} if bias else {}
    cas.cascade_shard_gemm(plan, cas.to_device(x, "bf16"), cas.to_device(w, "bf16"), guard[1:M + 1],
                           epilogue=cas.EPI_ROPE | (cas.EPI_BIAS if bias else 0), rope_cols=rot * d, head_dim=d,
                           rope_theta=500000.0, **kw)
    close(guard[1:M + 1], ref)
    assert (guard[0] == 7.0).all() and (guard[M + 1] == 7.0).all()


@pytest.mark.parametrize("M,N,K,launches", [(1, 3072, 4096, 2), (33, 1024, 2048, 2), (64, 3072, 1600, 2), (1, 3072, 1536, 1),
                                            (32, 1024, 768, 1), (4, 6144, 4096, 1)])
def test_narrow_outputs_of_long_reductions_are_rotated_behind(cas, M, N, K, launches):  # noqa: F811
    import torch
    x, w, y = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((M, K), (N, K), (M, N)))
    plan = cas.cascade_plan_create(M, 1, 1, np.zeros(1, np.int32))
    names = kernels_of(lambda: cas.cascade_shard_gemm(plan, x, w, y, epilogue=cas.EPI_ROPE, rope_cols=N // 2, head_dim=128,
                                                      rope_theta=10000.0))
    assert len(names) == launches and "gemm_rows_kernel" in names[0]


@pytest.mark.parametrize("M,K,kernel", [(4, 64, None), (64, 2048, None), (100, 128, "rope_vec_kernel")])
def test_angles_at_large_positions(cas, M, K, kernel):  # noqa: F811
    """Rows of X pick columns of W, so that what is rotated is exact; one rounding of the result (2^-9) and the angle are left."""
    import torch
    H, d = 4, 128
    rng = np.random.default_rng(M)
    pos = rng.integers(1 << 23, 1 << 24, M).astype(np.int32)
    plan = cas.cascade_plan_create(1, M, 1, np.zeros(M, np.int32), positions=pos)
    w = draw(rng, (H * d, K))
    x, wd = cas.to_device(np.eye(M, K, dtype=np.float32), "bf16"), cas.to_device(w, "bf16")
    y = torch.empty((M, H * d), dtype=torch.bfloat16, device="cuda")
    names = kernels_of(lambda: cas.cascade_shard_gemm(plan, x, wd, y, epilogue=cas.EPI_ROPE, rope_cols=H * d, head_dim=d, rope_theta=500000.0))
    assert (kernel is None and len(names) <= 2) or kernel in names[-1]
    v = w[:, :M].T.astype(np.float64)
    for h in range(H):
        ref = orc.rope(v[:, h * d:(h + 1) * d], pos, 500000.0)
        length = np.hypot(ref[:, :d // 2], ref[:, d // 2:])
        got = y[:, h * d:(h + 1) * d].float().cpu().numpy()
        assert (np.abs(got - ref) <= 2.0 ** -8 * np.concatenate([length, length], 1)).all()


@pytest.mark.parametrize("tokens,d_model,kernel", [(20, 256, "gemm_rows_kernel"), (200, 256, "gemm2_kernel"), (90, 3072, "splitk_heads_kernel")])
def test_table_of_a_layer_at_large_positions(cas, tokens, d_model, kernel):  # noqa: F811
    """The norm kernel's table of cos and sin, read by the few-row GEMM, the tiles and the sum of parts: the layer's keys."""
    import torch
    cfg = CONFIGS["C3"].with_(name="far", d_model=d_model, n_heads=4, n_kv_heads=2, head_dim=64, d_ff=256, batch=1, seq_len=tokens,
                              n_shards=1, index=76)
    a, h, w = np.zeros(tokens, np.int32), make_hidden(cfg), make_layer_weights(cfg)
    pos = np.random.default_rng(tokens).integers(1 << 23, 1 << 24, tokens).astype(np.int32)
    plan = cas.cascade_plan_create(1, tokens, 1, a, positions=pos)
    desc = cas.make_layer_desc(cfg)
    t = {k: cas.to_device(v, "bf16") for k, v in w.items()}
    hd, wts = cas.to_device(h, "bf16"), cas.make_layer_weights(t)
    out, ws = torch.empty_like(hd), cas.new_workspace(cas.cascade_layer_workspace_bytes(plan, desc))
    names = kernels_of(lambda: cas.cascade_layer_forward(plan, desc, wts, hd, out, ws))
    assert any(kernel in n for n in names[:3]) and not any("rope_" in n for n in names)
    kc = torch.zeros((1, 2, 1, tokens, 64), dtype=torch.bfloat16, device="cuda")
    cas.cascade_layer_kv_to_cache(plan, desc, ws, kc, kc.clone(), torch.zeros((1, 1), dtype=torch.int32, device="cuda"))
    w64 = {k: v.astype(np.float64) for k, v in w.items()}
    x = orc.norm(h[0].astype(np.float64), cfg.norm, w64["norm1_g"], None, cfg.eps)
    for g in range(2):
        ref = orc.rope(orc.linear(x, w64["wk"][g * 64:(g + 1) * 64]), pos, cfg.rope_theta)
        close(kc[0, g, 0], ref)
