"""Partial attention of head dimension 64 on either side of the choice between 4- and 8-wavefront workgroups (short
key/value shards, launches that leave CUs idle, neither) for one, two and four heads per workgroup, against the float64
oracle (the checks of test_gpu_parity)."""
import pytest

from test_gpu_parity import attn_case, cas, check_partials  # noqa: F401  (fixture and the oracle comparison)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv_heads", [(6, 6), (8, 4), (16, 4)])
@pytest.mark.parametrize("tokens,shards,mask", [(1000, 8, "causal"), (1100, 1, "causal"), (1100, 2, "none"), (1500, 4, "causal"),
                                                (1300, 5, "none")])
def test_partials(cas, heads, kv_heads, tokens, shards, mask):  # noqa: F811
    _, got, ref, _ = attn_case(cas, "bf16", 1, heads, kv_heads, tokens, 64, shards, "ragged", "packed", mask_kind=mask, seed=tokens)
    check_partials("bf16", got, ref)
