"""bf16 shard GEMM, epilogues that store from the accumulators: rows scattered and residual rows gathered through the plan's map
where a tile holds several sequences, outputs and residuals that start on 8-byte boundaries only, odd numbers of column
blocks per wavefront, last columns inside a lane's eight; several tiles per workgroup.  Against the float64 oracle."""
import numpy as np
import pytest

from cascade_inputs import make_assignment, round_to_bf16
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


# 128 x 96 (three column blocks per wavefront), 128 x 128 with one and two workgroups per CU, 192 and 256 columns; 100-row sequences
@pytest.mark.parametrize("batch,N,K", [(3, 192, 128), (3, 132, 192), (3, 200, 64), (41, 768, 768), (45, 2308, 768), (21, 6152, 2048),
                                       (41, 4104, 2048)])
@pytest.mark.parametrize("epi", ["plain", "residual", "bias_gelu", "bias_residual"])
@pytest.mark.parametrize("offset", [0, 4])
def test_rows_and_alignment(cas, batch, N, K, epi, offset):
    import torch
    n = 100
    M = batch * n
    rng = np.random.default_rng(N + batch)
    plan = cas.cascade_plan_create(batch, n, 5, make_assignment("ragged", n, 5, 3))
    perm = np.argsort(make_assignment("ragged", n, 5, 3), kind="stable")
    rows = (np.arange(batch)[:, None] * n + perm).ravel()                      # original row of every packed one
    x, w = draw(rng, (M, K)), draw(rng, (N, K), K ** -0.5)
    b, r = draw(rng, (N,), 0.3), draw(rng, (M, N))
    check = np.unique(np.concatenate([np.arange(0, M, 37), np.arange(M - 3, M)]))   # packed rows compared in float64
    ref = orc.linear(x[check].astype(np.float64), w.astype(np.float64))
    ep = 0
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
    cas.cascade_shard_gemm(plan, cas.to_device(x, "bf16"), cas.to_device(w, "bf16"), y, bias=cas.to_device(b, "bf16"), residual=res,
                           epilogue=ep, y_rows=cas.ROWS_ORIGINAL, res_rows=cas.ROWS_ORIGINAL)
    got = y.float().cpu().numpy()[rows[check]]
    assert np.abs(got - ref).max() / np.abs(ref).max() < TOL
    assert (out[:8 + offset] == 7.0).all() and (out[8 + offset + M * N:] == 7.0).all()
