"""The prefill kernels on rows whose last k step is half (K padded to an odd multiple of 64) and on the plain bit order: the k
loop split over waves, 64 x 128 and 128 x 128 tiles, 128 x 192 tiles of long rows, with int32 output and residual.  Bit for bit against
an exact integer product, with the last row and column ends that the loads of the half step must stay inside."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K", [(65, 130, 64), (129, 257, 192), (300, 515, 2999), (70, 128, 128), (64, 1, 1), (700, 2000, 192), (1000, 1500, 256),
                                   (200, 96, 448), (640, 2048, 576), (2600, 3300, 4160), (2600, 3300, 4096),
                                   (2600, 2700, 320), (2700, 2600, 64), (2561, 2689, 256), (2570, 2700, 1100)])
def test_half_steps_and_layouts(bl, layout, M, N, K):
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    W = torch.randint(-1, 2, (N, K), generator=g, device=DEV, dtype=torch.int8)
    Kp = bl.bl_padded_k(K)
    q = torch.zeros((M, Kp), dtype=torch.int8, device=DEV)
    q[:, :K] = torch.randint(-127, 128, (M, K), generator=g, device=DEV).to(torch.int8)
    scale = torch.rand(M, generator=g, device=DEV) * 0.01 + 1e-3
    rowsum = q.to(torch.int32).sum(1, dtype=torch.int32)
    packed, beta = bl.bl_pack_ternary(W, layout, beta=0.03125)
    want = (q[:, :K].double() @ W.double().t()).to(torch.int32)
    c = beta * scale
    y_want = want.to(torch.float32) * c[:, None]
    _, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_acc=False, K=K)
    assert torch.equal(y, y_want)
    acc, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, None, N, K=K)
    assert torch.equal(acc, want) and torch.equal(y, y_want)
    if K == Kp:
        res = torch.randn((M, N), generator=g, device=DEV)
        _, y = bl.bl_gemm_w158a8_res(packed, beta, layout, q, scale, rowsum, N, res)
        assert torch.equal(y, res + y_want)
