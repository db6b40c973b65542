"""Partials whose workgroups walk several key/value shards against the kernel that takes one shard at a time, bit for bit: the
latter runs positions of 2^30 and more, and partials depend on the order of the positions only.  Sizes on either side of
tiles, of the choice of wavefronts and of the shards per workgroup; empty, invisible and singleton shards; two shardings;
packed, original and strided rows; non-finite keys and values."""
import numpy as np
import pytest

from cascade_inputs import make_assignment
from launched import kernels_of
from test_gpu_parity import cas  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def both_paths(cas, B, H, Hkv, N, d, a, kv=None, mask="causal", layout="packed", token_major=False, u_mode=None, spoil=False,  # noqa: F811
               seed=0):
    """The bits of m, e and u for positions 0 .. N - 1 and for the same positions from 2^30 on."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    heads = torch.randn((B, N, H + 2 * Hkv, d), device="cuda", generator=g).bfloat16()
    if spoil:                                              # late keys and values that few queries see
        heads[:, N - 3, H:] = float("inf")
        heads[:, N // 2, H:] = float("nan")
    q, k, v = heads[:, :, :H], heads[:, :, H:H + Hkv], heads[:, :, H + Hkv:]
    strides = {}
    if token_major:
        row = (H + 2 * Hkv) * d
        strides = {"q_strides": (N * row, d, row), "kv_strides": (N * row, d, row)}
    else:
        q, k, v = (t.transpose(1, 2).contiguous() for t in (q, k, v))
    S = int((a if kv is None else kv).max()) + 1
    out = []
    for first in (0, 1 << 30):
        pos = np.arange(first, first + N, dtype=np.int64).astype(np.int32)
        kind = cas.MASK_CAUSAL if mask == "causal" else cas.MASK_NONE
        if kv is None:
            plan = cas.cascade_plan_create(B, N, S, a, positions=pos, mask_kind=kind)
        else:
            plan = cas.cascade_plan_create_rs(B, N, int(a.max()) + 1, a, S, kv, positions=pos, mask_kind=kind)
        m, e = (torch.full((B, H, S, N), 7.0, device="cuda") for _ in range(2))
        u = torch.full((B, S, H, N, d), 7.0, device="cuda")
        ws = cas.new_workspace(cas.cascade_partial_attn_workspace_bytes(plan, q, H, Hkv, d))
        names = kernels_of(lambda: cas.cascade_partial_attn(
            plan, q, k, v, m, e, u, H, Hkv, d, d ** -0.5, row_layout=cas.ROWS_PACKED if layout == "packed" else cas.ROWS_ORIGINAL,
            u_mode=cas.U_UNNORMALISED if u_mode is None else u_mode, workspace=ws, **strides))
        assert ("attn_bf16_kernel" if first else "attn_partial_kernel") in names[-1]
        torch.cuda.synchronize()
        out.append([t.view(torch.int32) for t in (m, e, u)])
    for x, y in zip(*out):
        assert torch.equal(x, y)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Hkv", [(3, 3), (4, 2), (8, 2), (8, 1)])
@pytest.mark.parametrize("N,beta,kind", [(1, 1, "contiguous"), (31, 3, "ragged"), (65, 1, "contiguous"), (129, 2, "perm"), (257, 40, "ragged"),
                                         (640, 5, "contiguous"), (1100, 3, "ragged"), (1300, 9, "perm")])
def test_same_bits_as_one_shard_at_a_time(cas, d, H, Hkv, N, beta, kind):  # noqa: F811
    for mask, layout in (("causal", "packed"), ("none", "original")):
        both_paths(cas, 2, H, Hkv, N, d, make_assignment(kind, N, beta, 3), mask=mask, layout=layout, seed=N + d)


@pytest.mark.parametrize("d,heads,N,beta", [(64, 24, 2048, 8), (64, 24, 1000, 16), (128, 16, 2048, 16), (128, 4, 4096, 4)])
def test_launches_of_several_rounds(cas, d, heads, N, beta):  # noqa: F811
    both_paths(cas, 2, heads, heads // 2, N, d, make_assignment("perm", N, beta, 5), seed=d)


@pytest.mark.parametrize("d", [64, 128])
def test_forms_of_the_call(cas, d):  # noqa: F811
    a = make_assignment("ragged", 700, 6, 9)
    both_paths(cas, 2, 8, 2, 700, d, a, layout="original", token_major=True, seed=1)
    both_paths(cas, 1, 4, 4, 700, d, a, u_mode=cas.U_NORMALISED, seed=2)
    both_paths(cas, 1, 4, 2, 700, d, a, spoil=True, seed=3)
    both_paths(cas, 1, 4, 2, 700, d, a, mask="none", spoil=True, seed=4)
    skewed = np.where(np.arange(3000) < 2900, 0, 1 + np.arange(3000) % 30).astype(np.int32)     # one long shard, many short ones
    both_paths(cas, 1, 4, 2, 3000, d, skewed, seed=5)
    both_paths(cas, 1, 6, 6, 700, d, a, kv=(a * 2 + np.arange(700) % 2).astype(np.int32), layout="original", seed=6)
