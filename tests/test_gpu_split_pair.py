"""Reductions split in two: two workgroups per 256 x 256 tile, half of K each, the first to finish hands its accumulators
to the second through scratch in the workspace.  Layers whose shapes select that on 256 CUs (9 x 12 tiles: not a
multiple of the 8 XCDs, the last row and column of tiles nearly empty; uneven halves in the FFN down projection),
against the float64 oracle, and what the exchange must not depend on."""
import numpy as np
import pytest

from cascade_inputs import CONFIGS, make_assignment, make_hidden, make_layer_weights
from oracle import cascade_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 results: a handful of 2^-9 roundings on the output's scale

# o projection over 80 heads of 128 (K = 10240, 160 k-tiles), FFN down over 10304 (161)
PAIR = CONFIGS["C3"].with_(name="pair-llama", d_model=2824, n_heads=80, n_kv_heads=2, head_dim=128, d_ff=10304, seq_len=2100,
                           n_shards=3, index=69)
# the flag words of a post-norm layer are cleared behind its o projection, which therefore leaves two planes
POST = PAIR.with_(name="pair-post", n_heads=81, n_kv_heads=3, norm_placement="post", bias=True, norm="layernorm", act="gelu",
                  rope=False, index=70)


@pytest.fixture(scope="module")
def cas():
    import torch
    import paper_2507_05228_amd as cas
    cas.load_library()
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("tile counts chosen for 256 CUs")
    return cas


def scratch_bytes(cas, cfg, tokens):
    """What the layer workspace holds besides the buffers of every layer: the scratch of the split reductions."""
    cfg = cfg.with_(seq_len=tokens, n_shards=1)
    plan = cas.cascade_plan_create(1, tokens, 1, np.zeros(tokens, np.int32))
    total = cas.cascade_layer_workspace_bytes(plan, cas.make_layer_desc(cfg, cas.ATTN_FUSED))
    H, Hkv, d = cfg.n_heads, cfg.n_kv_heads, cfg.head_dim
    rows = [2 * cfg.d_model, 2 * (H + 2 * Hkv) * d, 2 * H * d, 2 * cfg.d_model, 2 * cfg.d_ff, 4 * d if cfg.rope else 0]
    sizes = [tokens * r for r in rows] + [2 * Hkv * d * -(-tokens // 64) * 64, 2 * Hkv * d * tokens]       # V^T and K
    return total - sum(-(-s // 256) * 256 for s in sizes)


def test_shapes_take_two_parts(cas):
    flags = 2 * 256 * 4                                               # a ticket and a flag word for up to 256 tiles
    planes = 2 * 2100 * 2824 * 4                                      # more than the slots of 9 x 12 tiles
    assert scratch_bytes(cas, PAIR, 2100) == planes + flags and planes > 9 * 12 * 256 * 256 * 4
    assert scratch_bytes(cas, PAIR.with_(n_heads=8, d_ff=10176), 2100) == 0       # the limit on K
    assert scratch_bytes(cas, PAIR.with_(n_heads=8), 2824) == 0                   # 144 tiles: no two parts


@pytest.mark.parametrize("cfg", [PAIR, POST], ids=lambda c: c.name)
def test_layer(cas, cfg):
    a = make_assignment("ragged", cfg.seq_len, cfg.n_shards, 83)
    w, h = make_layer_weights(cfg), make_hidden(cfg)
    out = cas.layer_forward_numpy(cfg, w, h, a)
    ref = orc.layer_direct_batch(h, w, cfg)
    assert np.abs(out - ref).max() / np.abs(ref).max() < TOL


def test_same_bits_whatever_the_workspace_held_and_from_a_graph(cas):
    import torch
    cfg = PAIR
    plan = cas.cascade_plan_create(1, cfg.seq_len, cfg.n_shards, make_assignment("ragged", cfg.seq_len, cfg.n_shards, 83))
    desc = cas.make_layer_desc(cfg, cas.ATTN_FUSED)
    t = {k: cas.to_device(v, cfg.dtype) for k, v in make_layer_weights(cfg).items()}
    wts, h_in = cas.make_layer_weights(t), cas.to_device(make_hidden(cfg), cfg.dtype)
    ws = cas.new_workspace(cas.cascade_layer_stack_workspace_bytes(plan, desc, 2))
    outs = []
    for fill in (0xFF, None, 0x00, None):
        if fill is not None:
            ws.fill_(fill)
        outs.append(torch.empty_like(h_in))
        cas.cascade_layer_forward(plan, desc, wts, h_in, outs[-1], ws)
        torch.cuda.synchronize()
    assert all(torch.equal(o, outs[0]) for o in outs[1:])
    two, second = torch.empty_like(h_in), torch.empty_like(h_in)
    cas.cascade_layer_stack_forward(plan, desc, [wts, wts], h_in, two, ws)
    cas.cascade_layer_forward(plan, desc, wts, outs[0], second, ws)
    torch.cuda.synchronize()
    assert torch.equal(two, second)
    h_out = torch.empty_like(h_in)
    step = lambda: cas.cascade_layer_forward(plan, desc, wts, h_in, h_out, ws)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for rep in range(3):
        h_out.fill_(7.0)
        ws.fill_(0xA5 if rep % 2 else 0x00)
        junk = torch.randn(256, 256, device="cuda") @ torch.randn(256, 256, device="cuda")           # eager work in between
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(h_out, outs[0]), rep
