"""Norm kernels: a wavefront per row (up to two 16-byte pieces per lane) and a workgroup per row, at the edges of their pieces and
with rows that do not fill a workgroup; fp32 attention with eight wavefronts per query tile up to 32 head dimensions.  Against the float64 oracle."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights, round_to_bf16
from launched import layer_kernels
from oracle import cascade_oracle as orc

pytestmark = pytest.mark.gpu
TOL = {"bf16": 2e-2, "f32": 1e-5}                # one rounding to bf16; fp32 sums of a row


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


@pytest.mark.parametrize("dtype,D", [("bf16", 8), ("bf16", 512), ("bf16", 520), ("bf16", 768), ("bf16", 1024), ("bf16", 1032),
                                     ("bf16", 2056), ("f32", 4), ("f32", 256), ("f32", 260), ("f32", 512), ("f32", 516)])
@pytest.mark.parametrize("rows", [1, 3, 4, 9])
@pytest.mark.parametrize("kind", ["layernorm", "layernorm_bias", "rmsnorm"])
def test_rows_and_widths(cas, dtype, D, rows, kind):
    import torch
    rng = np.random.default_rng(D + rows)
    draw = lambda shape, mean: (rng.standard_normal(shape).astype(np.float32) + np.float32(mean))
    x, g, b = draw((rows, D), 0.5), draw((D,), 1.0), draw((D,), 0.0)
    if dtype == "bf16":
        x, g, b = (round_to_bf16(t) for t in (x, g, b))
    x64 = x.astype(np.float64)
    c = x64 if kind == "rmsnorm" else x64 - x64.mean(-1, keepdims=True)
    ref = c / np.sqrt((c * c).mean(-1, keepdims=True) + 1e-5) * g
    if kind == "layernorm_bias":
        ref = ref + b
    X = cas.to_device(x, dtype)
    Y = torch.full((rows + 2, D), 7.0, dtype=X.dtype, device="cuda")
    cas.cascade_norm(X, cas.to_device(g, dtype), cas.to_device(b, dtype) if kind == "layernorm_bias" else None, Y[1:rows + 1],
                     cas.NORM_RMSNORM if kind == "rmsnorm" else cas.NORM_LAYERNORM, 1e-5)
    got = Y[1:rows + 1].float().cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() / max(1.0, np.abs(ref).max()) < TOL[dtype]
    assert (Y[0] == 7.0).all() and (Y[rows + 1] == 7.0).all()


@pytest.mark.parametrize("dtype,D", [("f32", 260), ("f32", 388), ("f32", 512), ("bf16", 512), ("bf16", 520), ("bf16", 768), ("bf16", 1024)])
def test_a_wavefront_adds_a_row_in_the_order_of_a_workgroup(cas, dtype, D):
    """Rows four times as wide, zeros behind, which take a workgroup each: a quarter of the mean square, twice the result, both
    exact in binary, if the squares are added in the same order."""
    import torch
    rng = np.random.default_rng(D)
    x = rng.standard_normal((1000, D)).astype(np.float32) * np.exp(rng.uniform(-3, 3, (1000, D)).astype(np.float32))
    X = torch.zeros(1000, 4 * D, device="cuda", dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    X[:, :D] = cas.to_device(x, "f32")
    g = torch.ones(4 * D, device="cuda", dtype=X.dtype)
    narrow, wide = torch.empty_like(X[:, :D].contiguous()), torch.empty_like(X)
    cas.cascade_norm(X[:, :D].contiguous(), g[:D], None, narrow, cas.NORM_RMSNORM, 1e-5)
    cas.cascade_norm(X, g, None, wide, cas.NORM_RMSNORM, 1e-5 / 4)
    assert torch.equal(wide[:, :D], 2 * narrow)


@pytest.mark.parametrize("D", [64, 256, 260, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("kind", ["layernorm", "rmsnorm"])
def test_bias_is_added_before_the_one_rounding(cas, D, kind):
    """fp32: the product with the gain is not rounded on its own, in any column."""
    import torch
    rng = np.random.default_rng(D)
    x, g, b = (cas.to_device(rng.standard_normal(shape).astype(np.float32), "f32") for shape in ((200, D), (D,), (D,)))
    kind = cas.NORM_RMSNORM if kind == "rmsnorm" else cas.NORM_LAYERNORM
    scaled, out = torch.empty_like(x), torch.empty_like(x)
    cas.cascade_norm(x, torch.ones_like(g), None, scaled, kind, 1e-5)
    cas.cascade_norm(x, g, b, out, kind, 1e-5)
    assert torch.equal(out, (scaled.double() * g.double() + b.double()).float())


@pytest.mark.parametrize("batch,tokens", [(1, 64), (1, 65), (1, 81), (2, 127), (1, 129), (2, 258), (4, 513)])
@pytest.mark.parametrize("head_dim", [16, 20, 32, 64])
def test_fp32_attention_of_eight_wavefronts(cas, batch, tokens, head_dim):
    cfg = CONFIGS["C1"].with_(name="eight", d_model=4 * head_dim, n_heads=4, n_kv_heads=4, head_dim=head_dim, d_ff=64, batch=batch,
                              seq_len=tokens, n_shards=3, index=71)
    a = make_assignment("ragged", tokens, 3, 1)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a)
    ref = orc.layer_direct_batch(h, w, cfg)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL["f32"]
    # more than 32 head dimensions have no registers for it (20 to 40 % slower with spills)
    (name,) = (k for k in layer_kernels(cas, cfg, w, h, a) if "attn_f32_mfma_kernel" in k)
    assert ("Li8E" in name) == (tokens > 64 and head_dim <= 32 and -(-tokens // 16) * 4 * batch <= 256)
