"""KV-cache decode: shard capacities on either side of the one- / four-wavefront choice, few and many shards, ragged
lengths (empty, one row, full), against the float64 oracle (the checks of test_gpu_decode)."""
import pytest

from test_gpu_decode import cas, run_case  # noqa: F401  (fixture and the oracle comparison)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cap", [95, 96, 130, 255, 256])
def test_capacity_edges(cas, dtype, cap):  # noqa: F811
    lens = [[cap, 0, 1, cap - 1, 64], [1, cap, 17, 0, cap // 2]]
    run_case(cas, dtype, 2, 8, 2, 64, lens, cap)
