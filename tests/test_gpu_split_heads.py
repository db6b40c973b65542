"""q/k/v projection as a reduction split over several workgroups per tile, finished by a kernel that adds the planes and the
bias and rotates: layers whose shapes select 2 to 8 parts on 256 CUs, weights fused and apart, with and without rotation and
bias, ragged last tiles, several sequences, against the float64 oracle (the partials show q and k, the layer's output v)."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights
from launched import layer_kernels, split_tiles
from oracle import cascade_oracle as orc
from test_gpu_parity import cas  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 results: a handful of 2^-9 roundings on the output's scale

LLAMA = CONFIGS["C3"].with_(name="heads-llama", d_model=3072, n_heads=8, n_kv_heads=2, head_dim=64, d_ff=256, n_shards=3, index=71)
GPT = LLAMA.with_(name="heads-gpt", d_model=2048, n_heads=5, n_kv_heads=5, head_dim=128, bias=True, norm="layernorm", act="gelu",
                  rope=False, index=72)
WIDE = LLAMA.with_(name="heads-wide", d_model=2048, n_heads=16, n_kv_heads=4, head_dim=128, bias=True, index=73)


def splits(*args, **kw):
    return any("splitk_heads_kernel" in n for n in layer_kernels(*args, **kw))


@pytest.mark.parametrize("batch,tokens", [(1, 33), (1, 128), (2, 70), (1, 260)])
@pytest.mark.parametrize("base,placement", [(LLAMA, "pre"), (GPT, "pre"), (GPT, "post"), (WIDE, "pre")], ids=["llama", "gpt", "post", "wide"])
def test_layer(cas, base, placement, batch, tokens):  # noqa: F811
    cfg = base.with_(batch=batch, seq_len=tokens, norm_placement=placement)
    a = make_assignment("ragged", tokens, 3, 2)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    pos = (5 * np.arange(tokens) + 3).astype(np.int32)
    ref = orc.layer_direct_batch(h, w, cfg, positions=pos)
    for fused in (True, False):
        out, (m, e, _) = cas.layer_forward_numpy(cfg, w, h, a, positions=pos, attn_mode=cas.ATTN_MATERIALISED, return_partials=True,
                                                 fused_qkv=fused)
        assert np.abs(out - ref).max() / np.abs(ref).max() < TOL
        if fused:
            first = (m, e)
        else:               # one segment or three: the same sums in the same order
            assert np.array_equal(first[0], m) and np.array_equal(first[1], e)
    # three rows of tiles of 3072 columns are 72 tiles: not split
    assert splits(cas, cfg, w, h, a) == (base is not WIDE or tokens < 260)
    n = -(-3120 // (batch * tokens))                       # as many sequences as no shape here splits
    many = cfg.with_(batch=n * batch), w, np.concatenate([h] * n), a
    whole = cas.layer_forward_numpy(*many, positions=pos)[:batch]
    assert not splits(cas, *many)
    assert np.abs(out - whole).max() / np.abs(whole).max() < TOL


def test_256_wide_tiles(cas):  # noqa: F811
    """K = 8192 and 160 tiles of 128 x 128: six parts of 256 x 256."""
    import torch
    cfg = CONFIGS["C5"].with_(name="heads-256", d_ff=256, seq_len=150, n_shards=3, index=74)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    a = make_assignment("perm", 150, 3, 4)
    out = cas.layer_forward_numpy(cfg, w, h, a, fused_qkv=True)
    ref = orc.layer_direct_batch(h, w, cfg)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL
    names = layer_kernels(cas, cfg, w, h, a, fused_qkv=True)
    assert split_tiles(names)[0] == (256, 256)
    torch.cuda.empty_cache()


@pytest.mark.parametrize("d_model,heads,tokens,split", [(1024, 16, 33, False), (1024, 16, 128, False), (2048, 16, 17, False),
                                                        (2048, 16, 32, False), (2048, 16, 33, True), (1536, 8, 64, True), (4096, 16, 17, True)])
def test_only_where_the_second_launch_is_earned(cas, d_model, heads, tokens, split):  # noqa: F811
    """Columns: 3072 (16 heads of 64, keys and values as many) and 1536."""
    cfg = LLAMA.with_(d_model=d_model, n_heads=heads, n_kv_heads=heads, seq_len=tokens, batch=1)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    assert splits(cas, cfg, w, h, make_assignment("ragged", tokens, 3, 2)) == split
