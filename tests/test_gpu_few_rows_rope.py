"""Shard GEMM of few rows with the rotary epilogue (angles computed in the GEMM): row blocks of 16 and the 64-row limit,
several sequences, large positions, bias, columns behind the rotated ones, head dimensions it takes (32 .. 256) and the ones
that stay with the pass behind the GEMM (48, a last head cut short).  Against the float64 oracle."""
import numpy as np
import pytest

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
