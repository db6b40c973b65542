"""Fused attention without a mask, walked as one shard in packed order: the split walk (short shards at any size, single rounds)
and the unsplit one, last tiles from one row to full, key/value partitions of their own, positions that must not matter.
Against the float64 oracle."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights
from launched import layer_kernels
from oracle import cascade_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 results: a handful of 2^-9 roundings on the output's scale


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


def config(heads, kv_heads, head_dim, batch, tokens, shards):
    return CONFIGS["C3"].with_(name="unmasked", d_model=128, n_heads=heads, n_kv_heads=kv_heads, head_dim=head_dim, d_ff=128,
                               batch=batch, seq_len=tokens, n_shards=shards, sigma=0.1, index=68)


@pytest.mark.parametrize("heads,kv_heads", [(3, 3), (4, 2), (4, 1)])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("batch,tokens,shards", [(1, 32, 2), (1, 33, 2), (2, 64, 3), (1, 65, 1), (3, 127, 5), (1, 129, 4), (2, 320, 6),
                                                 (1, 390, 2), (40, 200, 8), (40, 257, 1)])
def test_layer(cas, heads, kv_heads, head_dim, batch, tokens, shards):
    """The last two: more workgroups than CUs, short shards and one of 257 tokens."""
    cfg = config(heads, kv_heads, head_dim, batch, tokens, shards)
    a = make_assignment("ragged", tokens, shards, 5)
    pos = np.random.default_rng(tokens).permutation(2 * tokens)[:tokens].astype(np.int32)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a, positions=pos, mask_kind=cas.MASK_NONE)
    for b in range(0, batch, max(1, batch - 1)):
        ref = orc.layer_direct(h[b], w, cfg, positions=pos, mask_kind="none")
        assert np.abs(out[b] - ref).max() / np.abs(ref).max() < TOL


@pytest.mark.parametrize("tokens,shards", [(100, 3), (300, 1)])
def test_key_value_partition_of_its_own(cas, tokens, shards):
    cfg = config(4, 2, 64, 2, tokens, shards)
    a = make_assignment("ragged", tokens, shards, 5)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    kv = (np.arange(tokens) * 7 % 5).astype(np.int32)
    out = cas.layer_forward_numpy(cfg, w, h, a, mask_kind=cas.MASK_NONE, token_to_kv_shard=kv)
    for b in range(2):
        ref = orc.layer_direct(h[b], w, cfg, mask_kind="none")
        assert np.abs(out[b] - ref).max() / np.abs(ref).max() < TOL


@pytest.mark.parametrize("tokens,bad", [(100, 3), (200, 70), (200, 199)])
def test_nan_token_reaches_every_row_of_its_sequence(cas, tokens, bad):
    cfg = config(3, 3, 64, 2, tokens, 4)
    a = make_assignment("ragged", tokens, 4, 5)
    w, h = make_layer_weights(cfg), make_hidden(cfg).copy()
    h[0, bad] = np.nan
    out = cas.layer_forward_numpy(cfg, w, h, a, mask_kind=cas.MASK_NONE)
    assert np.isnan(out[0]).any(-1).all() and np.isfinite(out[1]).all()


@pytest.mark.parametrize("heads,kv_heads,head_dim,batch,tokens,shards,kernel", [
    (3, 3, 64, 1, 33, 1, "attn_bf16"), (3, 3, 64, 1, 64, 1, "attn_bf16"), (3, 3, 64, 1, 65, 1, "attn_fused"), (4, 2, 128, 2, 64, 1, "attn_bf16"),
    (3, 3, 64, 86, 65, 1, "attn_bf16"), (3, 3, 64, 85, 65, 1, "attn_fused"), (3, 3, 128, 86, 128, 1, "attn_fused"), (3, 3, 64, 86, 128, 1, "attn_bf16"),
    (3, 3, 64, 86, 129, 1, "attn_fused"), (4, 2, 64, 65, 128, 2, "attn_bf16"), (4, 1, 64, 130, 64, 2, "attn_bf16"), (3, 3, 64, 90, 64, 2, "attn_fused")])
def test_short_shards_that_are_not_put_together_keep_their_kernel(cas, heads, kv_heads, head_dim, batch, tokens, shards, kernel):
    """On 256 CUs; shards of equal size."""
    cfg = config(heads, kv_heads, head_dim, batch, tokens, shards)
    a = (np.arange(tokens) % shards).astype(np.int32)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a, mask_kind=cas.MASK_NONE)
    for b in range(0, batch, max(1, batch - 1)):
        ref = orc.layer_direct(h[b], w, cfg, mask_kind="none")
        assert np.abs(out[b] - ref).max() / np.abs(ref).max() < TOL
    names = layer_kernels(cas, cfg, w, h, a, mask_kind=cas.MASK_NONE)
    assert [kernel in n for n in names if "attn_" in n] == [True]
