"""Split reductions in 192 x 256 tiles (two rows of tiles, columns that end inside a tile, uneven parts of K): layers whose FFN
down selects them on 256 CUs, against the float64 oracle."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights
from launched import layer_kernels, split_tiles
from oracle import cascade_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 results: a handful of 2^-9 roundings on the output's scale

WIDE = CONFIGS["C3"].with_(name="split-192", d_model=3720, n_heads=4, n_kv_heads=2, head_dim=128, d_ff=8256, n_shards=3, index=69)


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


@pytest.mark.parametrize("batch,tokens", [(1, 257), (1, 383), (2, 192)])
@pytest.mark.parametrize("placement", ["pre", "post"])
def test_layer(cas, batch, tokens, placement):
    cfg = WIDE.with_(batch=batch, seq_len=tokens, norm_placement=placement)
    a = make_assignment("ragged", tokens, 3, 2)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a)
    ref = orc.layer_direct_batch(h, w, cfg)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL
    assert split_tiles(layer_kernels(cas, cfg, w, h, a)) == [(128, 128), (192, 256)]       # o projection, FFN down
