"""Fused attention of causal layers in one round of workgroups: the split walk in position order for one, two and four
heads per workgroup, from two key/value tiles down to one, against the float64 oracle; positions not in token order."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights
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
