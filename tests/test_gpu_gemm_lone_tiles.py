"""Prefill products of 161 to 264 tiles of 64 x 128, one to a unit or a few more, whose rows are long (64 x 128 tiles, one product 128 x
128): ragged edges, half last k steps, both layouts and every set of outputs, bit for bit."""
import pytest

from test_gpu_gemm_routes import _product

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K", [(512, 2688, 2304), (512, 2561, 2240), (512, 4096, 2303), (1000, 1999, 2368), (129, 9999, 2560), (64, 32700, 4097),
                                   (512, 4097, 2560)])
def test_long_rows(bl, layout, M, N, K):
    packed, beta, q, scale, rowsum, want, y_want = _product(bl, layout, M, N, K)
    for _ in range(2):
        _, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_acc=False, K=K)
        assert torch.equal(y, y_want)
    acc, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, None, N, K=K)
    assert torch.equal(acc, want) and torch.equal(y, y_want)
    if K % 64 == 0:
        residual = torch.randn((M, N), generator=torch.Generator(device="cuda:0").manual_seed(3), device="cuda:0")
        acc, y = bl.bl_gemm_w158a8_res(packed, beta, layout, q, scale, rowsum, N, residual, want_acc=True)
        assert torch.equal(acc, want) and torch.equal(y, residual + y_want)
