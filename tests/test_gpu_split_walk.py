"""Fused attention of causal layers in one round of workgroups: the split walk in position order for one, two and four
heads per workgroup, from two key/value tiles down to one, against the float64 oracle; positions not in token order."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights, round_to_bf16
from oracle import cascade_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 results: a handful of 2^-9 roundings on the output's scale


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


@pytest.mark.parametrize("heads,kv_heads", [(3, 3), (4, 2), (4, 1), (6, 1)])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("batch,tokens,shards", [(1, 33, 2), (2, 64, 3), (1, 65, 1), (3, 127, 5), (1, 129, 4), (2, 257, 6), (1, 400, 3)])
def test_layer(cas, heads, kv_heads, head_dim, batch, tokens, shards):
    cfg = CONFIGS["C3"].with_(name="walk", d_model=128, n_heads=heads, n_kv_heads=kv_heads, head_dim=head_dim, d_ff=128,
                              batch=batch, seq_len=tokens, n_shards=shards, sigma=0.1, index=66)
    a = make_assignment("ragged", tokens, shards, 5)
    pos = np.random.default_rng(tokens).permutation(2 * tokens)[:tokens].astype(np.int32)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a, positions=pos)
    ref = orc.layer_direct_batch(h, w, cfg, positions=pos)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL


def attention_output(cas, q, k, v, a, shards, scale=None):
    """FUSED causal attention of bf16 values q [N, H, d], k, v [N, Hkv, d] as they are (token order): a post-norm layer
    whose projections select columns of its input, and the merged attention output it leaves in its workspace."""
    import torch
    N, H, d = q.shape
    Hkv = k.shape[1]
    D = (H + 2 * Hkv) * d
    cfg = CONFIGS["C3"].with_(name="select", d_model=D, n_heads=H, n_kv_heads=Hkv, head_dim=d, d_ff=64, batch=1, seq_len=N,
                              n_shards=shards, rope=False, norm_placement="post", index=67)
    eye = np.eye(D, dtype=np.float32)
    w = {"wq": eye[:H * d], "wk": 2 * eye[H * d:(H + Hkv) * d], "wv": eye[(H + Hkv) * d:], "wo": np.zeros((D, H * d), np.float32),
         "w_up": np.zeros((64, D), np.float32), "w_gate": np.zeros((64, D), np.float32), "w_down": np.zeros((D, 64), np.float32),
         "norm1_g": np.ones(D, np.float32), "norm2_g": np.ones(D, np.float32)}
    h = np.concatenate([q.reshape(N, -1), k.reshape(N, -1) / 2, v.reshape(N, -1)], 1).astype(np.float32)[None]
    plan = cas.cascade_plan_create(1, N, shards, a)
    desc = cas.make_layer_desc(cfg, cas.ATTN_FUSED, scale=scale)
    tensors = {n: cas.to_device(t, "bf16") for n, t in w.items()}
    h_in = cas.to_device(h, "bf16")
    h_out = torch.empty_like(h_in)
    ws = cas.new_workspace(cas.cascade_layer_workspace_bytes(plan, desc))
    cas.cascade_layer_forward(plan, desc, cas.make_layer_weights(tensors), h_in, h_out, ws)
    torch.cuda.synchronize()
    o = cas.cascade_layer_attention_output(plan, desc, ws, 1, H, d).float().cpu().numpy().astype(np.float64)
    out = np.empty_like(o)
    out[orc.shard_plan(a, shards)[1]] = o                                          # packed rows back to token order
    return out.reshape(N, H, d)


@pytest.mark.parametrize("heads,kv_heads,tokens", [(3, 3, 200), (4, 2, 200), (4, 1, 200), (4, 1, 300)])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("bad", [40, 100])
def test_infinite_key_is_not_seen_by_earlier_queries(cas, heads, kv_heads, tokens, head_dim, bad):
    """One element of the key at position `bad` is infinite (the first tile of either wavefront group): the outputs of
    the positions before it are those of a finite key, but for roundings of P and of the output that may fall the other
    way (2^-8 at most each): an infinite score makes its workgroup repeat the pass from moved offsets."""
    rng = np.random.default_rng(tokens + head_dim)
    draw = lambda n: round_to_bf16(rng.standard_normal((tokens, n, head_dim)).astype(np.float32))
    q, k, v = draw(heads), draw(kv_heads), draw(kv_heads)
    a = make_assignment("ragged", tokens, 3, 5)
    clean = attention_output(cas, q, k, v, a, 3)
    k = k.astype(np.float64)
    k[bad, :, 7] = 6e38                                                             # half of it is a bf16 number, it is not
    got = attention_output(cas, q, k, v, a, 3)
    worst = np.abs(got[:bad] - clean[:bad]).max()
    assert worst < 4 * 2.0 ** -8 * np.abs(v).max()
    assert np.isfinite(clean).all()


@pytest.mark.parametrize("heads,kv_heads", [(3, 3), (4, 2), (4, 1)])
@pytest.mark.parametrize("head_dim,tokens,shards", [(64, 60, 3), (128, 60, 3), (64, 200, 7), (128, 250, 10)])
def test_scores_of_short_shards_keep_the_bits_of_q(cas, heads, kv_heads, head_dim, tokens, shards):
    """A key has one element, in one of 16 columns, so that a score is one product, of up to 60.  Rounding the scaled
    query to bf16 once more would move it by up to 60 * 2^-8 = 0.23, another amount for every column, and the weights by as
    much; with the scale applied in fp32 what is left are the roundings of P and of the output (2^-8 at most each), and none
    where a query sees one key."""
    rng = np.random.default_rng(tokens + head_dim + heads)
    q, k = np.zeros((tokens, heads, head_dim), np.float32), np.zeros((tokens, kv_heads, head_dim), np.float32)
    scale = 1.0 / 3.0
    q[:, :, :16] = rng.uniform(12.0, 13.4, (tokens, heads, 16))
    np.put_along_axis(k, rng.integers(0, 16, (tokens, kv_heads, 1)), rng.uniform(12.0, 13.4, (tokens, kv_heads, 1)), 2)
    q, k = round_to_bf16(q), round_to_bf16(k)
    v = round_to_bf16(rng.standard_normal((tokens, kv_heads, head_dim)).astype(np.float32))
    a = make_assignment("ragged", tokens, shards, 5)
    got = attention_output(cas, q, k, v, a, shards, scale=scale)
    rep = heads // kv_heads
    for h in range(heads):
        s = q[:, h].astype(np.float64) @ k[:, h // rep].astype(np.float64).T * scale
        s[np.triu_indices(tokens, 1)] = -np.inf
        p = np.exp(s - s.max(1, keepdims=True))
        ref = (p / p.sum(1, keepdims=True)) @ v[:, h // rep].astype(np.float64)
        worst = np.abs(got[:, h] - ref).max()
        assert worst < 2 * 2.0 ** -8 * np.abs(v).max()
        assert (got[0, h] == v[0, h // rep]).all()
