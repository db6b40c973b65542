"""o projection and FFN down as reductions split over several workgroups per tile, finished (with the norm behind
them) by a row kernel: layers whose shapes select the split on 256 CUs, against the float64 oracle.  Ragged last tiles
in rows and columns, uneven parts, several sequences, both norm placements, biases, both row orders, layer stacks."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights
from launched import layer_kernels, split_tiles
from oracle import cascade_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 results: a handful of 2^-9 roundings on the output's scale

LLAMA = CONFIGS["C3"].with_(name="parts-llama", d_model=1032, n_heads=8, n_kv_heads=2, head_dim=128, d_ff=2112, index=63)
GPT = LLAMA.with_(name="parts-gpt", d_model=776, n_heads=12, n_kv_heads=12, head_dim=64, d_ff=1536, bias=True, norm="layernorm",
                  act="gelu", rope=False, index=64)
DEEP = LLAMA.with_(name="parts-deep", d_model=2056, n_heads=4, d_ff=8256, seq_len=1400, n_shards=3, index=65)


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


@pytest.mark.parametrize("batch,tokens", [(1, 17), (1, 64), (2, 65), (1, 129), (3, 100), (1, 500)])
@pytest.mark.parametrize("base", [LLAMA, GPT], ids=["llama", "gpt"])
@pytest.mark.parametrize("placement", ["pre", "post"])
def test_layer(cas, base, batch, tokens, placement):
    cfg = base.with_(batch=batch, seq_len=tokens, n_shards=3, norm_placement=placement)
    a = make_assignment("ragged", tokens, 3, 2)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a)
    ref = orc.layer_direct_batch(h, w, cfg)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL


def test_long_reduction_in_256_wide_tiles(cas):
    a = make_assignment("perm", DEEP.seq_len, 3, 2)
    w, h = make_layer_weights(DEEP), make_hidden(DEEP)
    ref = orc.layer_direct_batch(h, w, DEEP)
    out = cas.layer_forward_numpy(DEEP, w, h, a)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL
    assert split_tiles(layer_kernels(cas, DEEP, w, h, a)) == [(256, 256)]                  # FFN down, four parts


@pytest.mark.parametrize("base", [LLAMA, GPT], ids=["llama", "gpt"])
def test_stack_equals_single_layers_whatever_the_workspace_held(cas, base):
    import torch
    cfg = base.with_(batch=2, seq_len=90, n_shards=4)
    plan = cas.cascade_plan_create(2, 90, 4, make_assignment("ragged", 90, 4, 3))
    desc = cas.make_layer_desc(cfg)
    t = {k: cas.to_device(v, "bf16") for k, v in make_layer_weights(cfg).items()}
    wts = cas.make_layer_weights(t)
    h = cas.to_device(make_hidden(cfg), "bf16")
    ws = cas.new_workspace(cas.cascade_layer_stack_workspace_bytes(plan, desc, 2))
    once, twice, stacked = (torch.empty_like(h) for _ in range(3))
    ws.fill_(0xFF)
    cas.cascade_layer_forward(plan, desc, wts, h, once, ws)
    cas.cascade_layer_forward(plan, desc, wts, once, twice, ws)
    ws.fill_(0x7F)
    cas.cascade_layer_stack_forward(plan, desc, [wts, wts], h, stacked, ws)
    torch.cuda.synchronize()
    assert torch.equal(stacked, twice)
