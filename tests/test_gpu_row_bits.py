"""bf16 shard GEMM: the bits of a row do not depend on its place among the rows of a call.  Every row tile adds the products of k in
the same order, so rows that change places (and tiles) take their results along, bit for bit."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cas():
    import paper_2507_05228_amd as cas
    cas.load_library()
    return cas


# launches that fill the CUs with every tile of the one-wavefront kernel, and some that do not; short and long reductions
@pytest.mark.parametrize("M,N,K", [(4096, 768, 768), (4096, 2304, 768), (4096, 3072, 768), (6000, 768, 3072), (700, 6144, 4096), (1024, 4096, 4096),
                                   (1344, 4096, 4096), (2048, 4096, 4096), (2048, 6144, 4096), (1000, 14336, 2048), (3400, 2048, 2048), (200, 768, 768)])
@pytest.mark.parametrize("epi", ["plain", "bias_gelu", "bias_residual", "swiglu"])
def test_rows_take_their_bits_along(cas, M, N, K, epi):
    import torch
    g = torch.Generator(device="cuda").manual_seed(M + N)
    draw = lambda *shape: torch.randn(*shape, generator=g, device="cuda").to(torch.bfloat16)
    x, w, up, b, r = draw(M, K), draw(N, K) * 0.02, draw(N, K) * 0.02, draw(N), draw(M, N)
    ep = {"plain": 0, "bias_gelu": cas.EPI_BIAS | cas.EPI_GELU_ERF, "bias_residual": cas.EPI_BIAS | cas.EPI_RESIDUAL, "swiglu": cas.EPI_SWIGLU}[epi]

    def run(x, r):
        y = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
        cas.cascade_shard_gemm(None, x, w, y, W_up=up if epi == "swiglu" else None, bias=b if "bias" in epi else None,
                               residual=r if "residual" in epi else None, epilogue=ep)
        return y
    first = run(x, r)
    for shift in (64, 128, 320):                           # into the next row tile of each height, and further
        assert torch.equal(run(x.roll(shift, 0), r.roll(shift, 0)).roll(-shift, 0), first)
