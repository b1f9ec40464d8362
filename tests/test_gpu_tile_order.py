"""The two tile orders of a prefill launch: a rectangle of tiles per XCD, or (where that loads the busiest compute
unit more) one banded sequence of which each XCD takes an eighth.  Shapes of the second kind whose last band is part
filled, for the 64 x 128 and 128 x 128 tiles, with deferred stores and both fused epilogues; every output against an exact
integer product."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


def _order(tiles_m, tiles_n, bm, K):
    """(rectangles per column of XCDs or 0, row tiles of a band): the launcher's rule."""
    gm = 1
    while gm < 8 and -(-tiles_m // gm) * bm * K > 3 << 19:
        gm *= 2
    band = -(-tiles_m // gm)
    rect, share = band * -(-tiles_n // (8 // gm)), (tiles_m * tiles_n + 7) // 8
    if (rect + 31) // 32 <= (share + 31) // 32:
        return gm, band
    bands = -(-tiles_m // max(1, (3 << 19) // (bm * K)))
    return 0, -(-tiles_m // bands)


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def _inputs(bl, layout, M, N, K):
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    W = torch.randint(-1, 2, (N, K), generator=g, device=DEV, dtype=torch.int8)
    q = torch.randint(-127, 128, (M, K), generator=g, device=DEV).to(torch.int8)
    scale = torch.rand(M, generator=g, device=DEV) * 0.01 + 1e-3
    packed, beta = bl.bl_pack_ternary(W, layout, beta=0.03125)
    want = (q.float() @ W.float().t()).to(torch.int32)             # (exact: |sum| <= 127 K < 2^24)
    assert 127 * K < 1 << 24
    return packed, beta, q, scale, q.to(torch.int32).sum(1, dtype=torch.int32), want, want.float() * (beta * scale)[:, None], g


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K,bm", [(2100, 1664, 1024, 64), (2140, 3712, 1024, 128), (2140, 3712, 1088, 128), (2140, 4992, 2048, 128), (2700, 4224, 3328, 128)])
def test_even_shares_with_a_part_filled_last_band(bl, layout, M, N, K, bm):
    gm, band = _order(-(-M // bm), -(-N // 128), bm, K)
    assert gm == 0 and band < -(-M // bm) and -(-M // bm) % band
    packed, beta, q, scale, rowsum, want, y_want, g = _inputs(bl, layout, M, N, K)
    _, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_acc=False)
    assert torch.equal(y, y_want)
    acc, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N)
    assert torch.equal(acc, want) and torch.equal(y, y_want)
    res = torch.randn((M, N), generator=g, device=DEV)
    _, y = bl.bl_gemm_w158a8_res(packed, beta, layout, q, scale, rowsum, N, res)
    assert torch.equal(y, res + y_want)


@pytest.mark.parametrize("kind", ["residual", "gate"])
@pytest.mark.parametrize("M,N,K", [(2140, 3712, 1024), (2140, 4992, 2048), (2700, 4224, 3328)])
def test_fused_epilogues_in_even_shares(bl, kind, M, N, K):
    gm, band = _order(-(-M // 128), N // 128, 128, K)
    assert gm == 0 and -(-M // 128) % band
    packed, beta, q, scale, rowsum, want, y_want, g = _inputs(bl, 1, M, N, K)
    if kind == "residual":
        res = torch.randn((M, N), generator=g, device=DEV)
        t = res + y_want
    else:
        res, r = None, torch.relu(y_want[:, :N // 2])
        t = (r * r) * y_want[:, N // 2:]
    xb, y = torch.empty(t.shape, dtype=torch.bfloat16, device=DEV), torch.empty_like(t)
    absmax = torch.zeros(M, device=DEV)
    bl.bl_gemm_w158a8_fused(packed, beta, 1, q, scale, rowsum, N, bl.BL_EPI_RESIDUAL if res is not None else bl.BL_EPI_RELU2_GATE,
                            xb, absmax, residual=res, y=y)
    assert torch.equal(y, t) and torch.equal(xb, t.to(torch.bfloat16))
    assert torch.equal(absmax, xb.float().abs().amax(1))
