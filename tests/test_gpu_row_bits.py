"""bf16 shard GEMM: the bits of a row do not depend on its place among the rows of a call.  Every row tile adds the products of k in
the same order, so rows that change places (and tiles) take their results along, bit for bit."""
import pytest

from cascade_inputs import CONFIGS, make_assignment

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


# launches that fill the CUs with every tile of the one-wavefront kernel, and some that do not; short and long reductions
@pytest.mark.parametrize("M,N,K", [(4096, 768, 768), (4096, 2304, 768), (4096, 3072, 768), (6000, 768, 3072), (700, 6144, 4096), (1024, 4096, 4096),
                                   (1344, 4096, 4096), (2048, 4096, 4096), (2048, 6144, 4096), (1000, 14336, 2048), (3400, 2048, 2048), (200, 768, 768), (333, 14336, 4096),
                                   (20, 4096, 4096), (40, 768, 3072)])
@pytest.mark.parametrize("epi", ["plain", "bias_gelu", "bias_gelu_residual", "bias_residual", "swiglu", "swiglu_residual"])
def test_rows_take_their_bits_along(cas, M, N, K, epi):
    import torch
    g = torch.Generator(device="cuda").manual_seed(M + N)
    draw = lambda *shape: torch.randn(*shape, generator=g, device="cuda").to(torch.bfloat16)
    x, w, up, b, r = draw(M, K), draw(N, K) * 0.02, draw(N, K) * 0.02, draw(N), draw(M, N)
    bits = {"plain": 0, "bias": cas.EPI_BIAS, "gelu": cas.EPI_GELU_ERF, "residual": cas.EPI_RESIDUAL, "swiglu": cas.EPI_SWIGLU}
    ep = sum(bits[part] for part in epi.split("_"))

    def run(x, r):
        y = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
        cas.cascade_shard_gemm(None, x, w, y, W_up=up if "swiglu" in epi else None, bias=b if "bias" in epi else None,
                               residual=r if "residual" in epi else None, epilogue=ep)
        return y
    first = run(x, r)
    for shift in (64, 128, 320):                           # into the next row tile of each height, and further
        assert torch.equal(run(x.roll(shift, 0), r.roll(shift, 0)).roll(-shift, 0), first)


# q/k/v rotated in the epilogue: a row's bits are the same in tiles inside the matrix and in the last ones, which check their range;
# without and with biases, one matrix and three
@pytest.mark.parametrize("batch,tokens", [(3, 333), (2, 700), (3, 1000), (7, 45), (2, 1100), (3, 2200)])
@pytest.mark.parametrize("bias,fused_qkv", [(False, True), (False, False), (True, True)])
def test_equal_sequences_of_a_batch(cas, batch, tokens, bias, fused_qkv):
    import torch
    cfg = CONFIGS["C3"].with_(name="bits", d_model=2048, n_heads=32, n_kv_heads=8, d_ff=256, batch=batch, seq_len=tokens, n_shards=3, bias=bias, index=72)
    QW, D, f = (cfg.n_heads + 2 * cfg.n_kv_heads) * cfg.head_dim, cfg.d_model, cfg.d_ff
    g = torch.Generator(device="cuda").manual_seed(tokens)
    draw = lambda *shape, std=0.02, mean=0.0: (torch.randn(*shape, generator=g, device="cuda") * std + mean).to(torch.bfloat16)
    w = {"wo": draw(D, 4096), "w_gate": draw(f, D), "w_up": draw(f, D), "w_down": draw(D, f), "norm1_g": draw(D, mean=1.0), "norm2_g": draw(D, mean=1.0)}
    split = (4096, 1024, 1024)
    w.update(zip(("wq", "wk", "wv"), draw(QW, D).split(split)))
    if bias:
        w.update(zip(("bq", "bk", "bv"), draw(QW, std=0.5).split(split)))
        w["bo"] = draw(D)
    if not fused_qkv:
        w = {k: v.clone() for k, v in w.items()}
    plan = cas.cascade_plan_create(batch, tokens, 3, make_assignment("ragged", tokens, 3, 2))
    desc = cas.make_layer_desc(cfg)
    h = draw(1, tokens, D, std=1.0).expand(batch, -1, -1).contiguous()
    out = torch.empty_like(h)
    cas.cascade_layer_forward(plan, desc, cas.make_layer_weights(w), h, out, cas.new_workspace(cas.cascade_layer_workspace_bytes(plan, desc)))
    assert torch.equal(out, out[:1].expand_as(out))
