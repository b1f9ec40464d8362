"""Prefill products of short and long rows with many tiles, bit for bit against an exact integer product: several tiles to a workgroup
(fp32 output alone, its stores before the next tile's k loop), and launches that are mostly output, with every set of outputs, rows that
start on whole and broken lines, half last k steps and both layouts."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def _product(bl, layout, M, N, K):
    g = torch.Generator(device=DEV).manual_seed(M + N + K + layout)
    W = torch.randint(-1, 2, (N, K), generator=g, device=DEV, dtype=torch.int8)
    q = torch.zeros((M, bl.bl_padded_k(K)), dtype=torch.int8, device=DEV)
    q[:, :K] = torch.randint(-127, 128, (M, K), generator=g, device=DEV).to(torch.int8)
    scale = torch.rand(M, generator=g, device=DEV) * 0.01 + 1e-3
    packed, beta = bl.bl_pack_ternary(W, layout, beta=0.03125)
    want = (q[:, :K].float() @ W.float().t()).to(torch.int32) if 127 * K < 1 << 24 else (q[:, :K].double() @ W.double().t()).to(torch.int32)
    return packed, beta, q, scale, q.to(torch.int32).sum(1, dtype=torch.int32), want, want.to(torch.float32) * (beta * scale)[:, None]


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K", [(2600, 3328, 192), (2600, 3328, 1088), (1100, 8200, 3136), (2600, 3300, 3100), (2600, 3328, 256), (2600, 3328, 1280),
                                   (2048, 7008, 192), (1100, 11200, 4160), (1100, 11200, 1100)])
def test_many_tiles(bl, layout, M, N, K):
    """fp32 output alone."""
    tiles = -(-M // 128) * -(-N // 128)
    assert tiles > 2 * torch.cuda.get_device_properties(0).multi_processor_count
    packed, beta, q, scale, rowsum, _, y_want = _product(bl, layout, M, N, K)
    for _ in range(2):
        _, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_acc=False, K=K)
        assert torch.equal(y, y_want)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K", [(512, 5400, 64), (700, 3500, 200), (1000, 3840, 256), (1000, 3840, 257), (2600, 2700, 1100), (2600, 3300, 64), (2600, 3300, 1000),
                                   (2600, 3300, 3072), (2600, 3300, 3073), (2300, 4000, 512), (2300, 4000, 513), (3000, 6000, 192), (3000, 6000, 256),
                                   (2048, 7000, 640), (2048, 7000, 641), (2048, 6999, 1152), (2048, 6999, 1153),
                                   (2048, 7040, 1024), (2048, 7040, 3072), (2048, 7040, 3073)])
def test_short_rows(bl, layout, M, N, K):
    """Every set of outputs."""
    packed, beta, q, scale, rowsum, want, y_want = _product(bl, layout, M, N, K)
    _, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_acc=False, K=K)
    assert torch.equal(y, y_want)
    acc, _ = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_y=False, K=K)
    assert torch.equal(acc, want)
    acc, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, None, N, K=K)
    assert torch.equal(acc, want) and torch.equal(y, y_want)
