"""KV-cache decode of 4 and 8 query heads per kv head in bf16 (scores on the matrix cores): shard lengths around the 16-row
steps and the two steps in flight, both sides of the one- / four-wavefront choice, empty shards, both forms of u; values
outside the valid rows are never seen.  Against the float64 oracle (the checks of test_gpu_decode)."""
import pytest
import torch

from launched import kernels_of
from test_gpu_decode import cas, run_case  # noqa: F401  (fixture and the oracle comparison)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,d", [(8, 2, 64), (8, 2, 128), (8, 1, 64), (16, 2, 128)])
@pytest.mark.parametrize("cap", [1, 16, 17, 119, 120, 224])
def test_step_edges(cas, H, Hkv, d, cap):  # noqa: F811
    lens = [[min(cap, n) for n in row] for row in ([15, 16, 17, 0, 1, cap], [31, 32, 33, 63, 65, cap - 1], [47, 48, 49, 111, 129, 0])]
    run_case(cas, "bf16", 3, H, Hkv, d, lens, cap)


@pytest.mark.parametrize("u_mode", ["unnorm", "norm"])
@pytest.mark.parametrize("cap", [40, 120])
def test_many_shards(cas, cap, u_mode):  # noqa: F811
    """1024 wavefronts and more: one per shard of up to 40 rows, four per shard of up to 120."""
    lens = [[(7 * b + 5 * k) % (cap + 1) for k in range(65)] for b in range(4)]
    run_case(cas, "bf16", 4, 16, 4, 64, lens, cap, u_mode=u_mode)


@pytest.mark.parametrize("H,cap", [(8, 40), (8, 130), (16, 40)])
def test_rows_behind_the_valid_ones_are_not_seen(cas, H, cap):  # noqa: F811
    """NaN in every row from a shard's length on changes no bit."""
    B, Hkv, S, d = 2, 2, 5, 128
    g = torch.Generator(device="cuda").manual_seed(7)
    q = torch.randn((B, H, d), device="cuda", generator=g).bfloat16()
    k, v = (torch.randn((B, Hkv, S, cap, d), device="cuda", generator=g).bfloat16() for _ in range(2))
    lens = torch.tensor([[0, 1, 17, cap - 1, cap], [16, 15, cap, 33, 2]], dtype=torch.int32, device="cuda")
    behind = torch.arange(cap, device="cuda")[None, None, None] >= lens[:, None, :, None]
    out = []
    for fill in (0.0, float("nan")):
        kf, vf = (torch.where(behind[..., None].expand_as(t), torch.full_like(t, fill), t) for t in (k, v))
        m, e, u = torch.empty((B, H, S), device="cuda"), torch.empty((B, H, S), device="cuda"), torch.empty((B, S, H, d), device="cuda")
        cas.cascade_decode_partial_attn(q, kf, vf, lens, m, e, u, d ** -0.5)
        out.append((m, e, u))
    for a, b in zip(*out):
        assert torch.equal(a, b) and not torch.isnan(a).any()


@pytest.mark.parametrize("dtype,H,Hkv,d,kernel", [("bf16", 8, 2, 64, "decode_attn_mfma_kernel"), ("bf16", 16, 2, 128, "decode_attn_mfma_kernel"),
                                                  ("bf16", 4, 2, 128, "decode_attn_kernel"), ("bf16", 8, 2, 32, "decode_attn_kernel"),
                                                  ("f32", 8, 2, 128, "decode_attn_kernel")])
def test_which_kernel(cas, dtype, H, Hkv, d, kernel):  # noqa: F811
    t = lambda *shape: torch.zeros(shape, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")  # noqa: E731
    q, k, v, lens = t(1, H, d), t(1, Hkv, 2, 20, d), t(1, Hkv, 2, 20, d), torch.full((1, 2), 20, dtype=torch.int32, device="cuda")
    m, e, u = torch.empty((1, H, 2), device="cuda"), torch.empty((1, H, 2), device="cuda"), torch.empty((1, 2, H, d), device="cuda")
    (name,) = kernels_of(lambda: cas.cascade_decode_partial_attn(q, k, v, lens, m, e, u, d ** -0.5))
    assert kernel in name
