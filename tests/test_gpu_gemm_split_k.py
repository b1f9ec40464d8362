"""The split k loop in both orders of its tiles (rows first, columns first), with shares of the XCDs that are whole lines and that start
inside one, last tiles of one row and one column, both layouts and every set of outputs.  Bit for bit."""
import pytest

from test_gpu_gemm_routes import _product

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


ACROSS = [(512, 1024, 2560), (408, 925, 3519), (2497, 321, 1920), (3931, 256, 4480)]
DOWN = [(395, 1600, 2176), (329, 1409, 1984), (128, 1793, 768), (65, 1, 64), (1, 4097, 128)]


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K", ACROSS + DOWN)
def test_orders(bl, layout, M, N, K):
    packed, beta, q, scale, rowsum, want, y_want = _product(bl, layout, M, N, K)
    _, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_acc=False, K=K)
    assert torch.equal(y, y_want)
    acc, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, None, N, K=K)
    assert torch.equal(acc, want) and torch.equal(y, y_want)
